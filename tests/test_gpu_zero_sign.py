"""Sums start at +0 on every route: a zero grid under negative weights, whose
products are all -0, gives +0 whatever lane width or kernel a launch picks, and
a batched run has the sign bits of the grid run alone."""
import pytest

import stencil_inputs as si
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


def _plan(stl, shape, d, r, T, dt, dims):
    w = -si.normalised_weights(omodel.K_points(shape, d, r), seed=7600 + r)
    return stl.Plan(shape, d, r, w, dims, T=T, dtype=dt, path="valu", boundary="periodic")


@pytest.mark.parametrize("dt", ["f64", "f32"])
@pytest.mark.parametrize("shape,d,r,T,dims", [
    ("star", 2, 2, 4, (4096, 4096)), ("box", 2, 3, 2, (2048, 4096)), ("star", 2, 1, 1, (70, 90)),
    ("star", 3, 1, 1, (40, 50, 60)), ("star", 3, 2, 2, (40, 50, 60)), ("star", 3, 3, 2, (40, 50, 60)),
    ("box", 3, 1, 3, (40, 50, 60)), ("box", 3, 1, 1, (512, 320, 256)), ("box", 3, 2, 1, (40, 50, 60))])
def test_sum_of_negative_zeros(stl, shape, d, r, T, dt, dims):
    import torch
    x = torch.zeros(dims, device="cuda", dtype=stl.torch_dtype(dt))
    p = _plan(stl, shape, d, r, T, dt, dims)
    for steps in (T, 2 * T + 1):
        y = torch.full_like(x, float("nan"))
        p.run(x, y, steps)
        torch.cuda.synchronize()
        assert torch.count_nonzero(y) == 0
        assert not torch.signbit(y).any(), steps


def test_batch_has_the_sign_bits_of_the_grid_alone(stl):
    """The narrow odd grid of the list takes other lanes than the wide one."""
    import torch
    dims = [(2048, 4096), (64, 71)]
    plans = [_plan(stl, "box", 2, 3, 1, "f64", d) for d in dims]
    ins = [torch.zeros(d, device="cuda", dtype=torch.float64) for d in dims]
    outs = [torch.full_like(x, float("nan")) for x in ins]
    stl.run_batch(plans, ins, outs, [1, 1])
    for p, x, y in zip(plans, ins, outs):
        alone = torch.full_like(x, float("nan"))
        p.run(x, alone, 1)
        torch.cuda.synchronize()
        assert torch.equal(y.view(torch.int64), alone.view(torch.int64))
