"""Segments of a pass (planes of the 3D row kernel, rows of the 2D kernel) on
grids whose swept axis is long: many of them, alone and beside small grids.
Tolerances as for the other VALU kernels: FP64 relative max-norm error <= 1e-12,
FP32 <= 1e-5."""
import pytest

from gpu_util import case_inputs, oracle, rel_inf, run_gpu

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


def _time(run, reps=5):
    """Shortest time of a call, ms."""
    import torch
    best = float("inf")
    for _ in range(reps):
        t0, t1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        t0.record()
        run()
        t1.record()
        torch.cuda.synchronize()
        best = min(best, t0.elapsed_time(t1))
    return best


@pytest.mark.parametrize("shape,r,T", [("star", 1, 1), ("box", 1, 1), ("star", 2, 1), ("star", 1, 2)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_tall_grid(stl, shape, r, T, dt):
    """9000 planes are swept at the rate of 3000 (one segment for all of them
    would take some 60 times as long), alone and in a batch beside a small
    grid, and have the oracle's values."""
    import torch
    plans, ins, outs = [], [], []
    for k, dims in enumerate([(9000, 20, 30), (3000, 20, 30), (40, 20, 30)]):
        u0, u0r, t, w = case_inputs(shape, 3, r, dims, dt, seed=7700 + k)
        plans.append(stl.Plan(shape, 3, r, w, dims, T=T, dtype=dt, path="valu", halo=0.5))
        ins.append(t.cuda())
        outs.append(torch.empty_like(ins[-1]))
        plans[-1].run(ins[-1], outs[-1], T)
        torch.cuda.synchronize()
        ref = oracle(shape, 3, r, w, u0, T, "dirichlet", 0.5)
        assert rel_inf(outs[-1].to(torch.float64).cpu().numpy(), ref) <= TOL[dt], dims
    steps = 20 * T
    tall, less = (_time(lambda: p.run(x, y, steps)) for p, x, y in list(zip(plans, ins, outs))[:2])
    assert tall <= 12 * less, (tall, less)
    alone = [y.clone() for y in outs]
    both = _time(lambda: stl.run_batch(plans[::2], ins[::2], outs[::2], [steps] * 2))
    assert both <= 12 * less, (both, less)
    assert torch.equal(outs[0], alone[0])


@pytest.mark.parametrize("shape,r,T", [("star", 1, 3), ("star", 2, 2), ("star", 3, 1), ("box", 1, 2)])
@pytest.mark.parametrize("dt", ["f64", "f32"])
def test_segments_of_one_to_three_planes(stl, shape, r, T, dt):
    for dims in [(7, 33, 70), (2, 20, 40), (12, 9, 130)]:
        u0, u0r, t, w = case_inputs(shape, 3, r, dims, dt, seed=7750 + dims[0])
        ref = oracle(shape, 3, r, w, u0, T, "periodic")
        for planes in (1, 2, 3):
            p = stl.Plan(shape, 3, r, w, dims, T=T, dtype=dt, path="valu", boundary="periodic", tile_rows=planes)
            assert rel_inf(run_gpu(p, t, T), ref) <= TOL[dt], (dims, planes)


def test_float64_lanes_within_the_registers(stl):
    """Box-2D3R float64 fused four deep keeps to lanes whose accumulators leave
    room for two waves per SIMD: a pass takes some 2.3 times one of T = 2 (2.75
    with four columns per lane and one wave)."""
    import torch
    dims = (8192, 8192)
    K = 49
    w = [1.0 / K] * K
    x = torch.rand(dims, device="cuda", dtype=torch.float64)
    y = torch.empty_like(x)
    ms = {}
    for T in (2, 4):
        p = stl.Plan("box", 2, 3, w, dims, T=T, dtype="f64", path="valu")
        p.run(x, y, 8 * T)
        ms[T] = _time(lambda: p.run(x, y, 8 * T))
    assert ms[4] <= 2.5 * ms[2], ms


@pytest.mark.parametrize("dt", ["f64", "f32", "f16"])
def test_very_wide_grid(stl, dt):
    """Rows of more bands than there are work items to deal out keep the wide
    lanes: 12 million columns take three times as long as 4 million (one-column
    lanes some ten times), with the oracle's values on windows."""
    import numpy as np
    import torch
    import stencil_inputs as si
    from gpu_util import U_STORE
    from oracle import core as ocore
    r, T, n0 = 3, 4, 5
    w = si.normalised_weights(13, seed=7800)
    u0, t = si.round_to(si.uniform_grid((n0, 12_000_000), seed=7810), dt)
    ms = []
    for n1 in (4_000_000, 12_000_000):
        x = t[:, :n1].contiguous().cuda()
        y = torch.empty_like(x)
        p = stl.Plan("star", 2, r, w, (n0, n1), T=T, dtype=dt, path="valu", halo=0.25)
        p.run(x, y, T)
        ms.append(_time(lambda: p.run(x, y, T)))
        for c in (0, n1 // 2, n1 - 16):
            ref = ocore.run_window("star", 2, r, w, u0[:, :n1], T, (0, c), (n0, c + 16), "dirichlet", 0.25)
            got = y[:, c:c + 16].to(torch.float64).cpu().numpy()
            tol = TOL[dt] if dt in TOL else U_STORE[dt] + 2 * T * 13 * 2.0 ** -24
            assert np.max(np.abs(got - ref)) <= tol, (n1, c)
    assert ms[1] <= 5 * ms[0], ms


def test_narrow_grid_beside_a_wide_one(stl):
    """A narrow grid with an odd row length, which only one-column lanes take,
    leaves a large grid of the same batch its wide lanes (the whole batch on
    one-column lanes takes 3.4 times as long); bits as alone."""
    import torch
    r, T, steps = 3, 4, 16
    w = [1.0 / 13] * 13
    plans, ins, outs, alone = [], [], [], []
    for k, dims in enumerate([(8192, 8192), (64, 71), (90, 41)]):
        plans.append(stl.Plan("star", 2, r, w, dims, T=T, dtype="f32", path="valu", boundary="periodic"))
        g = torch.Generator(device="cuda")
        g.manual_seed(7900 + k)
        ins.append(torch.rand(dims, generator=g, device="cuda"))
        outs.append(torch.empty_like(ins[-1]))
        alone.append(torch.empty_like(ins[-1]))
        plans[-1].run(ins[-1], alone[-1], steps)
    stl.run_batch(plans, ins, outs, [steps] * 3)
    one = _time(lambda: plans[0].run(ins[0], alone[0], steps))
    all_ = _time(lambda: stl.run_batch(plans, ins, outs, [steps] * 3))
    assert all_ <= 1.8 * one, (all_, one)
    for a, b in zip(alone, outs):
        assert torch.equal(a, b)


@pytest.mark.parametrize("shape,r,T,dims", [("star", 1, 2, (1, 131072, 131072)), ("star", 1, 1, (1, 131072, 131071))])
def test_planes_of_more_threads_than_a_launch_takes(stl, shape, r, T, dims):
    """A plane of 1.7e10 points (one column a lane makes 4.4e9 to 4.9e9 threads):
    windows at the corners and around the middle row and column against the
    oracle on blocks that hold what they depend on."""
    import torch
    import stencil_inputs as si
    if torch.cuda.mem_get_info()[0] < 180 << 30:
        pytest.skip("needs 140 GB of free device memory")
    w = si.normalised_weights(7, seed=8000)
    n0, n1, n2 = dims
    g = torch.Generator(device="cuda")
    g.manual_seed(8010)
    x = torch.rand(dims, generator=g, device="cuda", dtype=torch.float32)
    y = torch.full(dims, float("nan"), device="cuda", dtype=torch.float32)
    p = stl.Plan(shape, 3, r, w, dims, T=T, dtype="f32", path="valu", halo=0.25)
    p.run(x, y, T)
    torch.cuda.synchronize()
    m = r * T
    for cy in (0, n1 // 4, n1 // 2, n1):
        for cx in (0, n2 // 2, n2):
            lo = [max(cy - 20, 0), max(cx - 20, 0)]
            hi = [min(cy + 20, n1), min(cx + 20, n2)]
            a = [max(v - m, 0) for v in lo]
            e = [min(hi[0] + m, n1), min(hi[1] + m, n2)]
            block = x[:, a[0]:e[0], a[1]:e[1]].to(torch.float64).cpu().numpy()
            ref = oracle(shape, 3, r, w, block, T, "dirichlet", 0.25)
            ref = ref[:, lo[0] - a[0]:hi[0] - a[0], lo[1] - a[1]:hi[1] - a[1]]
            got = y[:, lo[0]:hi[0], lo[1]:hi[1]].to(torch.float64).cpu().numpy()
            assert rel_inf(got, ref) <= TOL["f32"], (cy, cx)
    assert not torch.isnan(y[0, ::4096, ::511]).any()
    del x, y
    torch.cuda.empty_cache()
