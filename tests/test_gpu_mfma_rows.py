"""16-bit matrix passes in the row layout at the edges of their tiles (48 x 128
points, or 80 x 256 on grids past the last-level cache): ragged last tiles,
rows of every residue modulo the 8-element chunk, frames that cross one or
several grid edges, and the Dirichlet band redone in one launch.  Absolute
error against the oracle on the storage-rounded data within the worst-case
bound of gpu_util.lowp_bound."""
import numpy as np
import pytest

import stencil_inputs as si
from gpu_util import case_inputs, lowp_bound, oracle, run_gpu
from oracle import core as ocore
from oracle import model as omodel

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def stl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_00477_amd as stl
    stl.lib()
    return stl


@pytest.mark.parametrize("shape,r,T", [("box", 2, 4), ("star", 2, 4), ("star", 3, 2), ("box", 1, 1), ("box", 1, 3)])
@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_tile_edges(stl, shape, r, T, dt, boundary):
    for dims in [(47, 127), (49, 129), (96, 256), (33, 40), (17, 300), (150, 131), (50, 1002), (64, 17), (200, 515)]:
        u0, u0r, t, w = case_inputs(shape, 2, r, dims, dt, seed=7100 + 10 * r + T + dims[1])
        p = stl.Plan(shape, 2, r, w, dims, T=T, dtype=dt, path="mfma", boundary=boundary, halo=0.5)
        got = run_gpu(p, t, 2 * T)
        ref = oracle(shape, 2, r, w, u0r, 2 * T, boundary, 0.5)
        bound = lowp_bound(dt, omodel.K_fused(shape, 2, r, T), 2, float(np.max(np.abs(u0r))))
        assert float(np.max(np.abs(got - ref))) <= bound, dims


@pytest.mark.parametrize("dims", [(8200, 8192), (8195, 8203)])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_large_tiles_on_windows(stl, dims, boundary):
    import torch
    shape, r, T, dt = "box", 2, 4, "bf16"
    w = si.normalised_weights(25, seed=7200)
    u0r, t = si.round_to(si.uniform_grid(dims, seed=7210), dt)
    x = t.cuda()
    y = torch.empty_like(x)
    p = stl.Plan(shape, 2, r, w, dims, T=T, dtype=dt, path="mfma", boundary=boundary, halo=0.25)
    p.run(x, y, T)
    torch.cuda.synchronize()
    bound = lowp_bound(dt, omodel.K_fused(shape, 2, r, T), 1, 1.0)
    n0, n1 = dims
    for lo in [(0, 0), (n0 - 20, n1 - 20), (n0 - 20, 0), (0, n1 - 20), (70, 246), (n0 // 2, n1 - 20), (4000, 4090)]:
        hi = (lo[0] + 20, lo[1] + 20)
        ref = ocore.run_window(shape, 2, r, w, u0r, T, lo, hi, boundary, 0.25)
        got = y[lo[0]:hi[0], lo[1]:hi[1]].to(torch.float64).cpu().numpy()
        assert float(np.max(np.abs(got - ref))) <= bound, lo
