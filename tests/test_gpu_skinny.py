"""GPU parity of layers over at most 64 tokens in the dense order, whose
forward and dX products take the few-rows kernel where it is the faster one
(tests/test_routes.py: which of them do, in every form of 16, 32 and 64 rows;
an fp32 dX over 1024 or more outputs keeps the plan's splits of K): one token
up to one past its limit, widths that are no whole number of 16 columns or
64-byte steps of K, and a K that the eight waves share unevenly; Y, dX and
every dG_k against the oracle.

Tolerance as for the layers: max |gpu - ref| / max |ref| <= 1e-4 (fp32),
<= 2e-2 (bf16).
"""
import pytest

from oracle import ttm as OT
from tests.gpu_util import TTMRun, rel_err, to_dev, to_np
from tests.test_gpu_ttm import TOL, _inputs

pytestmark = pytest.mark.gpu

SHAPES = [
    ((8, 8, 12), (16, 16, 12)),      # 768 -> 3072
    ((5, 8, 17), (3, 11, 24)),       # 680 -> 792: K of 21.25 / 42.5 steps, 49.5 column tiles
    ((10, 10, 10), (9, 11, 8)),      # 1000 -> 792
]


@pytest.mark.parametrize("act", ["f32", "bf16"])
@pytest.mark.parametrize("b", [1, 7, 16, 17, 32, 33, 64, 65])
@pytest.mark.parametrize("shape", SHAPES, ids=["768x3072", "680x792", "1000x792"])
def test_few_tokens(shape, b, act):
    n, m = shape
    r = (1, 6, 7, 1)
    print(f"skinny {shape} b={b} {act}", flush=True)
    cores, D, X, dY = _inputs(301 + b, n, m, r, b, act)
    Yr = OT.forward_dense(X, cores, D)
    dXr, dGr = OT.backward_dense(X, dY, cores, D)
    run = TTMRun(n, m, r, cores, D, b, act, force_order=0)
    Xt, dYt = to_dev(X, act), to_dev(dY, act)
    errs = {"Y": rel_err(to_np(run.forward(Xt)), Yr)}
    dX, dG = run.backward(Xt, dYt)
    errs["dX"] = rel_err(to_np(dX), dXr)
    for k in range(3):
        errs[f"dG{k}"] = rel_err(to_np(dG[k]), dGr[k])
    bad = {k: v for k, v in errs.items() if not v <= TOL[act]}
    assert not bad, bad
