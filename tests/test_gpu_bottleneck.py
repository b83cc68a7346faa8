"""GPU parity of the two-group sweep through one bond (first group without
output modes, second without input modes: the paper's TT layout) on its own
kernels: one to four cores per group, bond ranks on both sides of 16, 32 and
64 padding, rows that are no whole number of 128-byte lines or 64-column
strips, token counts around the 16-, 32- and 64-token tiles, several token
splits in the meets, compacted masks, unit modes, unaligned activations, calls
below the planned batch, with and without reuse; against the oracle.

Tolerances as for the layers: max |gpu - ref| / max |ref| <= 1e-4 (fp32),
<= 2e-2 (bf16: W's factors and the states are rounded to bf16 once each).
"""
import numpy as np
import pytest

from oracle import ttm as OT
from paper_2405_14377_amd import comera as C
from tests.gpu_util import TTMRun, rel_err, to_dev, to_np
from tests.test_gpu_ttm import TOL, _inputs

pytestmark = pytest.mark.gpu


def _layout(ins, outs, ranks):
    return tuple(ins) + (1,) * len(outs), (1,) * len(ins) + tuple(outs), (1,) + tuple(ranks) + (1,)


def _order(n, m, r, act, b, cut, mask_active=None):
    """Index of the left-to-right sweep with one cut after core cut - 1."""
    p = C.TTMPlan(n, m, r, C.BF16 if act == "bf16" else C.F32, batch=b, mask_active=mask_active)
    d = len(n)
    want = "sweep-lr [" + ",".join(map(str, range(cut))) + "][" + ",".join(map(str, range(cut, d))) + "]"
    i = [p.order_info(j)["desc"] for j in range(p.num_orders)].index(want)
    assert p.order_info(i)["executable"]
    return i


def _errors(run, X, dY, cores, D, act, Xt=None, dYt=None, b=None):
    Yr = OT.forward_dense(X, cores, D)
    dXr, dGr = OT.backward_dense(X, dY, cores, D)
    Xt = to_dev(X, act) if Xt is None else Xt
    dYt = to_dev(dY, act) if dYt is None else dYt
    Y = run.forward(Xt, b=b)
    dX, dG = run.backward(Xt, dYt, b=b)
    errs = {"Y": rel_err(to_np(Y), Yr), "dX": rel_err(to_np(dX), dXr)}
    for k, g in enumerate(dG):
        errs[f"dG{k}"] = rel_err(to_np(g), dGr[k])
    return {k: v for k, v in errs.items() if not v <= TOL[act]}, (Y, dX, dG)


SHAPES = [
    # (seed, ins, outs, ranks, b)
    (201, (8,), (16,), (5,), 1),                               # one core per group
    (202, (16, 8), (8, 24), (7, 16, 9), 17),
    (203, (8, 5, 8), (24, 8), (17, 33, 32, 20), 63),           # R = 32 -> one padded group of 32
    (204, (4, 6, 4, 3), (8, 4, 3, 2), (4, 12, 20, 33, 18, 9, 3), 129),   # four cores, R = 33 -> 64
    (205, (8, 8, 13), (11, 8, 8), (30, 64, 48, 64, 30), 300),  # 832 x 704: ragged lines and strips
    (206, (1, 8, 16), (16, 1, 40), (3, 6, 31, 5, 8), 2050),    # unit modes, two token splits
    (207, (8, 8, 12), (16, 16, 12), (30, 30, 24, 30, 30), 523),
]


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("case", SHAPES, ids=[f"s{c[0]}" for c in SHAPES])
def test_shapes(case, act):
    seed, ins, outs, ranks, b = case
    n, m, r = _layout(ins, outs, ranks)
    cores, D, X, dY = _inputs(seed, n, m, r, b, act)
    i = _order(n, m, r, act, b, len(ins))
    outs_ = []
    for reuse in (False, True):
        print(f"bottleneck {case} {act} reuse={reuse}", flush=True)
        run = TTMRun(n, m, r, cores, D, b, act, force_order=i, reuse=reuse)
        bad, out = _errors(run, X, dY, cores, D, act)
        assert not bad, bad
        outs_.append(out)
    for a, c in zip(outs_[0][:2], outs_[1][:2]):
        assert np.array_equal(to_np(a), to_np(c))
    for a, c in zip(outs_[0][2], outs_[1][2]):
        assert np.array_equal(to_np(a), to_np(c))


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("b", [8200, 16400])
def test_token_tiles(b, act):
    """Token counts that take the 32- and the 64-token tile."""
    n, m, r = _layout((8, 4), (4, 16), (6, 10, 6))
    cores, D, X, dY = _inputs(211, n, m, r, b, act)
    print(f"bottleneck tiles b={b} {act}", flush=True)
    run = TTMRun(n, m, r, cores, D, b, act, force_order=_order(n, m, r, act, b, 2))
    assert not _errors(run, X, dY, cores, D, act)[0]


@pytest.mark.parametrize("act", ["f32", "bf16"])
def test_masks_smaller_batch_and_unaligned(act):
    """Compacted masks with the mask gradients; fewer tokens than planned;
    activations that start off a 16-byte boundary (same bits as aligned)."""
    import torch
    n, m, r = _layout((4, 3, 4), (4, 4, 3), (4, 12, 40, 12, 4))
    b, plan_b = 133, 200
    rng = np.random.default_rng(221)
    cores, _, X, dY = _inputs(221, n, m, r, b, act, masks=None)
    active = [(rng.random(x) < 0.7).astype(np.uint8) for x in r[1:-1]]
    for a in active:
        a[0] = 1
    D = [a.astype(np.float32) * rng.uniform(0.5, 1.5, a.size).astype(np.float32) for a in active]
    ma = [int(x) for a in active for x in a]
    i = _order(n, m, r, act, plan_b, 3, ma)
    run = TTMRun(n, m, r, cores, D, plan_b, act, mask_active=ma, force_order=i)
    bad, (Y, dX, dG) = _errors(run, X, dY, cores, D, act, b=b)
    assert not bad, bad
    Xt, dYt = to_dev(X, act), to_dev(dY, act)
    dX2, dG2, dD = run.backward_masks(Xt, dYt, b=b)
    ref = OT.mask_grads_dense(X, dY, cores, D)
    scale = OT.mask_grad_term_scale(X, dY, cores, D)
    for k, g in enumerate(dD):
        on = active[k].astype(bool)
        got = to_np(g)
        assert np.all(got[~on] == 0.0), k
        s = np.max(np.abs(ref[k][on])) if act == "f32" else np.max(scale[k][on])
        assert np.max(np.abs(got[on] - ref[k][on])) <= TOL[act] * s, k
    _, _, dD2 = run.backward_masks(Xt, dYt, b=b, want_dg=False)
    for a, c in zip(dD, dD2):
        assert torch.equal(a, c)

    def shifted(t):
        buf = torch.zeros(t.numel() + 1, dtype=t.dtype, device=t.device)
        buf[1:] = t.reshape(-1)
        return buf[1:].reshape(t.shape)

    Xs, dYs = shifted(Xt), shifted(dYt)
    assert Xs.data_ptr() % 16 and dYs.data_ptr() % 16
    Ys, dXs = shifted(torch.zeros_like(Y)), shifted(torch.zeros_like(dX))
    dGs = [torch.empty_like(g) for g in run.G]
    C.comera_ttm_forward(run.plan.handle, b, Xs, run.G, run.D, Ys, run.ws)
    C.comera_ttm_backward(run.plan.handle, b, Xs, dYs, run.G, run.D, dXs, dGs, run.ws)
    assert torch.equal(Ys, Y) and torch.equal(dXs, dX)
    for a, c in zip(dGs, dG):
        assert torch.equal(a, c)


def test_partial_outputs():
    """dX only, dG only and a subset of dG."""
    import torch
    n, m, r = _layout((4, 4, 6), (6, 4, 4), (5, 6, 7, 6, 5))
    cores, D, X, dY = _inputs(231, n, m, r, 90, "f32")
    run = TTMRun(n, m, r, cores, D, 90, "f32", force_order=_order(n, m, r, "f32", 90, 3))
    dXr, dGr = OT.backward_dense(X, dY, cores, D)
    Xt, dYt = to_dev(X), to_dev(dY)
    assert rel_err(to_np(run.backward(Xt, dYt, want_dg=False)[0]), dXr) <= 1e-4
    for g, ref in zip(run.backward(Xt, dYt, want_dx=False)[1], dGr):
        assert rel_err(to_np(g), ref) <= 1e-4
    some = [None, torch.empty_like(run.G[1]), None, None, torch.empty_like(run.G[4]), None]
    C.comera_ttm_backward(run.plan.handle, 90, Xt, dYt, run.G, run.D, None, some, run.ws)
    for k in (1, 4):
        assert rel_err(to_np(some[k]), dGr[k]) <= 1e-4


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("where", ["X", "dY"])
@pytest.mark.parametrize("ranks", [(3, 1, 2), (6, 30, 7), (6, 33, 7)], ids=["R1", "R30", "R33"])
def test_infinities_stay_infinities(ranks, where, act):
    """One infinite activation among positive values and positive cores: every
    result it reaches is that infinity (a rank padded with zeros must not turn
    it into NaN), every other one is as finite as in the oracle."""
    n, m, r = _layout((4, 6), (8, 4), ranks)
    b = 72
    rng = np.random.default_rng(241)
    cores = [rng.uniform(0.5, 1.0, (r[k], m[k], n[k], r[k + 1])).astype(np.float32) for k in range(4)]
    X, dY = (rng.integers(1, 5, (b, w)).astype(np.float32) for w in (24, 32))
    (X if where == "X" else dY)[17, 9] = np.inf
    Yr = OT.forward_dense(X, cores)
    dXr, dGr = OT.backward_dense(X, dY, cores)
    run = TTMRun(n, m, r, cores, None, b, act, force_order=_order(n, m, r, act, b, 2))
    Xt, dYt = to_dev(X, act), to_dev(dY, act)
    got = [run.forward(Xt)]
    dX, dG = run.backward(Xt, dYt)
    for g, ref in zip(got + [dX] + dG, [Yr, dXr] + dGr):
        g, fin = to_np(g), np.isfinite(ref)
        assert not np.isnan(ref).any() and np.array_equal(np.isposinf(g), ~fin)
        if fin.any():
            assert rel_err(g[fin], ref[fin]) <= TOL[act]
