"""3D passes at the edges of their tiles: 64-column layouts less a skirt
of r*T columns per side, 4 or 8 waves of 4-6 rows less r*(T-1) rows per side,
segments from a few planes (small grids) up.  Tolerances as for the other VALU
kernels: FP64 relative max-norm error <= 1e-12, FP32 <= 1e-5."""
import numpy as np
import pytest

from gpu_util import case_inputs, oracle, rel_inf, run_gpu

pytestmark = pytest.mark.gpu

TOL = {"f64": 1e-12, "f32": 1e-5}
VARIANTS = [("star", 1, 2), ("star", 1, 3), ("star", 2, 2), ("star", 2, 3), ("star", 3, 2), ("box", 1, 2),
            ("box", 1, 3), ("star", 1, 1), ("star", 2, 1), ("star", 3, 1), ("box", 1, 1), ("box", 2, 1),
            ("box", 3, 1)]


@pytest.fixture(scope="module")
def stl():
    import torch
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2603_00477_amd as stl
    stl.lib()
    return stl


def edge_dims(r, T):
    """One tile exactly, one column / row more, fewer points than the skirt,
    and one plane only."""
    bx = 64 - 2 * r * T
    return [(7, 30, bx), (12, 33, bx + 1), (1, 3, 2 * bx - 1), (40, 2, 5), (2, 77, 130), (65, 64, 64)]


@pytest.mark.parametrize("shape,r,T", VARIANTS)
@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_rows3d_tile_edges(stl, shape, r, T, dt, boundary):
    for dims in edge_dims(r, T):
        u0, u0r, t, w = case_inputs(shape, 3, r, dims, dt, seed=6100 + 10 * r + T + sum(dims))
        for rows in (None, 5):  # planes per segment: chosen, and fixed with a ragged last one
            p = stl.Plan(shape, 3, r, w, dims, T=T, dtype=dt, path="valu", boundary=boundary, halo=0.5,
                         tile_rows=rows)
            got = run_gpu(p, t, T)
            ref = oracle(shape, 3, r, w, u0, T, boundary, 0.5)
            assert rel_inf(got, ref) <= TOL[dt], (dims, rows)


@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_rows3d_batch_of_uneven_grids(stl, dt):
    """A batched launch picks its waves and segments for the whole list: each
    result equals the grid swept alone, bit for bit."""
    import torch
    dims = [(97, 97, 97), (3, 5, 7), (64, 20, 131), (1, 61, 60), (30, 200, 200)]
    for shape, r, T in VARIANTS:
        plans, ins, outs, alone = [], [], [], []
        for k, d in enumerate(dims):
            u0, u0r, t, w = case_inputs(shape, 3, r, d, dt, seed=6300 + k)
            plans.append(stl.Plan(shape, 3, r, w, d, T=T, dtype=dt, path="valu",
                                  boundary="periodic" if k % 2 else "dirichlet", halo=0.25))
            ins.append(t.cuda())
            outs.append(torch.empty_like(ins[-1]))
            alone.append(torch.empty_like(ins[-1]))
        stl.run_batch(plans, ins, outs, [T] * len(dims))
        for p, x, y in zip(plans, ins, alone):
            p.run(x, y, T)
        torch.cuda.synchronize()
        for k in range(len(dims)):
            assert torch.equal(outs[k], alone[k]), (shape, r, T, dims[k])
            assert np.isfinite(outs[k].cpu().numpy()).all()


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("r", [2, 3])
def test_large_box_beyond_the_small_grid_rule(stl, dt, r):
    """Boxes r >= 2 over 160^3 points (float32 takes 32-row tiles there): ragged
    tiles and segments, sampled windows, and a batch with a small grid."""
    import torch
    from oracle import core as ocore
    import stencil_inputs as si
    w = si.normalised_weights((2 * r + 1) ** 3, seed=6500 + r)
    plans, ins, outs = [], [], []
    for k, dims in enumerate([(161, 165, 163), (9, 40, 33)]):
        u0 = si.uniform_grid(dims, seed=6510 + k)
        x = si.round_to(u0, dt)[1].cuda()
        p = stl.Plan("box", 3, r, w, dims, T=1, dtype=dt, path="valu", halo=0.25)
        y = torch.empty_like(x)
        p.run(x, y, 1)
        torch.cuda.synchronize()
        for lo in [(0, 0, 0), tuple(n - 6 for n in dims), tuple(min(n // 2, n - 6) for n in dims)]:
            hi = tuple(a + 6 for a in lo)
            ref = ocore.run_window("box", 3, r, w, u0, 1, lo, hi, "dirichlet", 0.25)
            got = y[tuple(slice(a, b) for a, b in zip(lo, hi))].cpu().numpy()
            assert rel_inf(got, ref) <= TOL[dt], (dims, lo)
        plans.append(p)
        ins.append(x)
        outs.append(y)
    batch = [torch.empty_like(y) for y in outs]
    stl.run_batch(plans, ins, batch, [1, 1])
    torch.cuda.synchronize()
    for a, b in zip(outs, batch):
        assert torch.equal(a, b)


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("r", [2, 3])
@pytest.mark.parametrize("boundary", ["dirichlet", "periodic"])
def test_large_box_segment_lengths(stl, dt, r, boundary):
    """The first and last 2r planes of a segment compute part of the weights:
    segments of one plane, of 2r (no full plane) and beyond, a ragged last one."""
    dims = (4 * r + 7, 33, 37)
    u0, u0r, t, w = case_inputs("box", 3, r, dims, dt, seed=6400 + r)
    ref = oracle("box", 3, r, w, u0, 1, boundary, 0.5)
    for planes in (1, 2, 2 * r, 2 * r + 1, 4 * r + 3, 4 * r + 7):
        p = stl.Plan("box", 3, r, w, dims, T=1, dtype=dt, path="valu", boundary=boundary, halo=0.5,
                     tile_rows=planes)
        assert rel_inf(run_gpu(p, t, 1), ref) <= TOL[dt], planes


@pytest.mark.parametrize("shape,r", [("star", 2), ("box", 1)])
def test_one_step_large_and_small_kernels_agree(stl, shape, r):
    """A one-step pass over a large grid of whole aligned rows takes the
    16-byte-load kernel; the same grid one column narrower does not.  Both
    hold the oracle's values on sampled windows, and a batch that mixes them
    with a small grid equals each run alone."""
    import torch
    from oracle import core as ocore
    import stencil_inputs as si
    K = 6 * r + 1 if shape == "star" else 27
    w = si.normalised_weights(K, seed=6400 + r)
    plans, ins, outs = [], [], []
    for k, dims in enumerate([(256, 512, 512), (256, 512, 511), (20, 30, 40)]):
        u0 = si.uniform_grid(dims, seed=6410 + k)
        x = si.round_to(u0, "f32")[1].cuda()
        p = stl.Plan(shape, 3, r, w, dims, T=1, dtype="f32", path="valu", boundary="periodic")
        y = torch.empty_like(x)
        p.run(x, y, 1)
        torch.cuda.synchronize()
        for lo in [(0, 0, 0), tuple(n - 6 for n in dims), tuple(min(n // 2, n - 6) for n in dims)]:
            hi = tuple(a + 6 for a in lo)
            ref = ocore.run_window(shape, 3, r, w, u0, 1, lo, hi, "periodic")
            got = y[tuple(slice(a, b) for a, b in zip(lo, hi))].cpu().numpy()
            assert rel_inf(got, ref) <= TOL["f32"], (dims, lo)
        plans.append(p)
        ins.append(x)
        outs.append(y)
    batch = [torch.empty_like(y) for y in outs]
    stl.run_batch(plans, ins, batch, [1, 1, 1])
    torch.cuda.synchronize()
    for a, b in zip(outs, batch):
        assert torch.equal(a, b)
