"""Outputs written over inputs of the same size, where a call reads each
token's row before it writes it: the same bits as into separate memory."""
import pytest

from tests.gpu_util import TTMRun, to_dev
from tests.test_gpu_ttm import _inputs
from paper_2405_14377_amd import comera as C

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("over", ["X", "dY"])
@pytest.mark.parametrize("b", [3, 40])
def test_fused_sweep_dx(b, over, act):
    """Small batches of the fused sweep, which otherwise give every output a
    workgroup of its own."""
    import torch
    n, m, r = (8, 8, 12), (12, 8, 8), (1, 8, 8, 1)
    cores, D, X, dY = _inputs(401 + b, n, m, r, b, act)
    order = C.TTMPlan(n, m, r, batch=b).num_orders - 1
    run = TTMRun(n, m, r, cores, D, b, act, force_order=order)
    Xt, dYt = to_dev(X, act), to_dev(dY, act)
    print(f"in place b={b} over {over} {act}", flush=True)
    dX, dG = run.backward(Xt, dYt)
    out = Xt if over == "X" else dYt
    dG2 = [torch.empty_like(g) for g in dG]
    C.comera_ttm_backward(run.plan.handle, b, Xt, dYt, run.G, run.D, out, dG2, run.ws)
    assert torch.equal(out, dX) and all(torch.equal(a, c) for a, c in zip(dG, dG2))


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("b", [1, 16, 40])
def test_forward_over_few_tokens(b, act):
    """Y over X where the product would otherwise take the few-rows kernel,
    whose workgroups all read all of X: split K, summed after the reads."""
    import torch
    n, m, r = (8, 8, 12), (12, 8, 8), (1, 6, 7, 1)
    cores, D, X, dY = _inputs(431 + b, n, m, r, b, act)
    run = TTMRun(n, m, r, cores, D, b, act, force_order=0)
    Xt = to_dev(X, act)
    Y = run.forward(Xt)
    print(f"forward in place b={b} {act}", flush=True)
    C.comera_ttm_forward(run.plan.handle, b, Xt, run.G, run.D, Xt, run.ws)
    # another order of the sums over K than the few-rows kernel's
    tol = 2e-2 if act == "bf16" else 1e-5
    assert (Xt.float() - Y.float()).abs().max() <= tol * Y.float().abs().max()
