"""2D VALU passes over the lane widths (1, 2 or 4 columns) and band layouts the
launcher picks between: rows that are no whole number of vectors (bands
anchored to both edges), narrow grids, unaligned buffers, and large grids
checked on sampled windows.  Tolerances as for the other VALU kernels (16-bit
storage: one rounding of the result per pass beside the inputs' own)."""
import numpy as np
import pytest

import stencil_inputs as si
from gpu_util import U_STORE, case_inputs, oracle, rel_inf, run_gpu
from oracle import core as ocore

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}


@pytest.fixture(scope="module")
def stl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_00477_amd as stl
    stl.lib()
    return stl


@pytest.mark.parametrize("shape,r,T", [("star", 1, 1), ("star", 3, 4), ("box", 2, 2), ("box", 3, 3), ("star", 1, 8),
                                       ("box", 7, 1)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_row_lengths(stl, shape, r, T, dt, boundary):
    """Row lengths on both sides of one band of each width and of every
    residue modulo the vector."""
    for dims in [(40, 63), (33, 130), (50, 255), (21, 257), (37, 498), (29, 1001), (35, 1002), (31, 1003)]:
        u0, u0r, t, w = case_inputs(shape, 2, r, dims, dt, seed=6600 + r + T + dims[1])
        p = stl.Plan(shape, 2, r, w, dims, T=T, dtype=dt, path="valu", boundary=boundary, halo=0.5)
        got = run_gpu(p, t, T)
        ref = oracle(shape, 2, r, w, u0, T, boundary, 0.5)
        assert rel_inf(got, ref) <= TOL[dt], dims


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16", "f16"])
@pytest.mark.parametrize("n1", [4096, 4097, 4098, 4099])
def test_large_grids_on_windows(stl, dt, n1):
    """Sizes at which the wider lanes are picked; a periodic and a Dirichlet
    pass, windows on the corners, the right edge and inside.  16-bit storage:
    float32 arithmetic on the rounded data, then one rounding (relative
    u_store of values below 1)."""
    import torch
    n0 = 2500
    for shape, r, T, boundary in [("star", 3, 4, "periodic"), ("box", 2, 2, "dirichlet")]:
        K = 4 * r + 1 if shape == "star" else (2 * r + 1) ** 2
        w = si.normalised_weights(K, seed=6700 + r)
        u0 = si.uniform_grid((n0, n1), seed=6710)
        u0r, t = si.round_to(u0, dt)
        p = stl.Plan(shape, 2, r, w, (n0, n1), T=T, dtype=dt, path="valu", boundary=boundary, halo=0.25)
        x = t.cuda()
        y = torch.empty_like(x)
        p.run(x, y, T)
        torch.cuda.synchronize()
        for lo in [(0, 0), (n0 - 12, n1 - 12), (100, n1 - 12), (n0 // 2, 236), (n0 - 12, 0), (777, n1 // 2)]:
            hi = (lo[0] + 12, lo[1] + 12)
            ref = ocore.run_window(shape, 2, r, w, u0r if dt in U_STORE and dt != "f32" else u0, T, lo, hi, boundary, 0.25)
            got = y[lo[0]:hi[0], lo[1]:hi[1]].to(torch.float64).cpu().numpy()
            if dt in TOL:
                assert rel_inf(got, ref) <= TOL[dt], (shape, lo)
            else:
                K_steps = T * K * 2.0 ** -24  # float32 accumulation of each step
                assert np.max(np.abs(got - ref)) <= U_STORE[dt] + 2 * K_steps, (shape, lo)


@pytest.mark.parametrize("dt", ["f64", "f32", "bf16"])
def test_unaligned_buffers(stl, dt):
    """Grids that start one element past an aligned address give the same
    bits as aligned ones (vectors move at element alignment)."""
    import torch
    for dims in [(64, 512), (301, 1213)]:
        w = si.normalised_weights(25, seed=6800)
        n = dims[0] * dims[1]
        x = torch.rand(n + 1, device="cuda").to(stl.torch_dtype(dt))
        y = torch.zeros_like(x)
        xa = x[1:].clone().reshape(dims)
        ya = torch.empty_like(xa)
        p = stl.Plan("box", 2, 2, w, dims, T=2, dtype=dt, path="valu", boundary="periodic")
        p.run(x[1:].reshape(dims), y[1:].reshape(dims), 5)
        p.run(xa, ya, 5)
        torch.cuda.synchronize()
        assert torch.equal(y[1:].reshape(dims), ya)
        assert float(y[0]) == 0.0


def test_batch_over_widths(stl):
    """A batched launch takes one width for its whole list (a narrow grid in
    it rules the wide lanes out): every result equals the grid run alone."""
    import torch
    lists = [[(3000, 4096), (2000, 4096)], [(3000, 4093), (64, 70)], [(1024, 1021), (7, 900), (900, 3)]]
    for shape, r, T in [("star", 2, 4), ("box", 3, 2)]:
        for k, dl in enumerate(lists):
            plans, ins, outs, alone = [], [], [], []
            for m, dims in enumerate(dl):
                w = si.normalised_weights(9 if shape == "star" else 49, seed=6900 + m)
                plans.append(stl.Plan(shape, 2, r, w, dims, T=T, dtype="f32", path="valu",
                                      boundary="periodic" if m % 2 else "dirichlet"))
                g = torch.Generator(device="cuda")
                g.manual_seed(6900 + 10 * k + m)
                ins.append(torch.rand(dims, generator=g, device="cuda"))
                outs.append(torch.full_like(ins[-1], float("nan")))
                alone.append(torch.empty_like(ins[-1]))
            stl.run_batch(plans, ins, outs, [2 * T + 1] * len(dl))
            for p, x, y in zip(plans, ins, alone):
                p.run(x, y, 2 * T + 1)
            torch.cuda.synchronize()
            for a, b, dims in zip(alone, outs, dl):
                assert torch.equal(a, b), (shape, dims)
