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


@pytest.mark.parametrize("shape,r,T", [("box", 2, 4), ("star", 2, 3), ("star", 3, 2), ("box", 1, 1), ("box", 3, 1)])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_tile_edges_compensated(stl, shape, r, T, boundary):
    """The compensated mode's own staging (32-byte chunks split into two frames)
    at the same edges, rows shorter than a chunk among them."""
    for dims in [(47, 127), (49, 129), (33, 40), (17, 300), (150, 131), (64, 17), (200, 515), (40, 7), (9, 3)]:
        if boundary == "periodic" and min(dims) < 2 * r * T + 1:
            continue
        u0, u0r, t, w = case_inputs(shape, 2, r, dims, "bf16x3", seed=7300 + 10 * r + T + dims[1])
        p = stl.Plan(shape, 2, r, w, dims, T=T, dtype="bf16x3", path="mfma", boundary=boundary, halo=0.5)
        got = run_gpu(p, t, 2 * T)
        ref = oracle(shape, 2, r, w, u0r, 2 * T, boundary, 0.5)
        umax = max(float(np.max(np.abs(u0r))), 0.5)
        bound = lowp_bound("bf16x3", omodel.K_fused(shape, 2, r, T), 2, umax)
        assert float(np.max(np.abs(got - ref))) <= bound, dims


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("shape,r,T", [("star", 3, 2), ("box", 1, 3), ("box", 1, 7)])
def test_large_tiles_of_other_composites(stl, dt, shape, r, T):
    import torch
    dims = (8117, 8203)
    K = omodel.K_points(shape, 2, r)
    w = si.normalised_weights(K, seed=7400 + r)
    u0r, t = si.round_to(si.uniform_grid(dims, seed=7410), dt)
    x = t.cuda()
    n0, n1 = dims
    for boundary in (["periodic"] if T == 7 else ["periodic", "dirichlet"]):
        y = torch.empty_like(x)
        p = stl.Plan(shape, 2, r, w, dims, T=T, dtype=dt, path="mfma", boundary=boundary, halo=0.25)
        p.run(x, y, T)
        torch.cuda.synchronize()
        bound = lowp_bound(dt, omodel.K_fused(shape, 2, r, T), 1, 1.0)
        for lo in [(0, 0), (n0 - 20, n1 - 20), (n0 - 20, 0), (0, n1 - 20), (70, 246), (4000, 4090)]:
            hi = (lo[0] + 20, lo[1] + 20)
            ref = ocore.run_window(shape, 2, r, w, u0r, T, lo, hi, boundary, 0.25)
            got = y[lo[0]:hi[0], lo[1]:hi[1]].to(torch.float64).cpu().numpy()
            assert float(np.max(np.abs(got - ref))) <= bound, (boundary, lo)


@pytest.mark.parametrize("dt", ["bf16", "f16"])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_batch_of_large_tiles_with_small_grids(stl, dt, boundary):
    """A batch that moves more than 256 MB takes the large tiles for its small
    ragged grids too: bits of the grids run alone, the small ones against the
    oracle."""
    import torch
    shape, r, T = "box", 2, 2
    w = si.normalised_weights(25, seed=7500)
    plans, ins, outs, alone, small = [], [], [], [], []
    for k, dims in enumerate([(8100, 8203), (37, 61), (130, 515), (90, 257)]):
        u0r, t = si.round_to(si.uniform_grid(dims, seed=7510 + k), dt)
        plans.append(stl.Plan(shape, 2, r, w, dims, T=T, dtype=dt, path="mfma", boundary=boundary, halo=0.25))
        ins.append(t.cuda())
        outs.append(torch.full_like(ins[-1], float("nan")))
        alone.append(torch.empty_like(ins[-1]))
        if k:
            small.append((k, u0r))
    stl.run_batch(plans, ins, outs, [2 * T] * 4)
    for p, x, y in zip(plans, ins, alone):
        p.run(x, y, 2 * T)
    torch.cuda.synchronize()
    for a, b in zip(alone, outs):
        assert torch.equal(a, b)
    bound = lowp_bound(dt, omodel.K_fused(shape, 2, r, T), 2, 1.0)
    for k, u0r in small:
        ref = oracle(shape, 2, r, w, u0r, 2 * T, boundary, 0.25)
        assert float(np.max(np.abs(outs[k].to(torch.float64).cpu().numpy() - ref))) <= bound, k
