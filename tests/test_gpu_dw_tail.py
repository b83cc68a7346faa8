"""GPU parity of dW = X^T dY on the straight-to-LDS kernels when the token
count does not fill the last K stage (64 tokens in bf16, 32 in fp32): one
token, one token less than a stage, an odd number in between, token counts
whose last split holds only the short stage, a product of less than a stage
in all, and splits on the other side of the rule, which the bounds-checked
kernel takes (tests/test_routes.py checks which).  Dense order; every dG_k
against the oracle (a row counted twice or left out shows as an error far
above the tolerance: each token weighs about 1 / sqrt(b) of dW).

Tolerance as for the layers: max |gpu - ref| / max |ref| <= 1e-4 (fp32) and,
dG being fp32 sums of exact bf16 products, the same bound in bf16.
"""
import pytest

from oracle import ttm as OT
from tests.gpu_util import TTMRun, rel_err, to_dev, to_np
from tests.test_gpu_ttm import _inputs

pytestmark = pytest.mark.gpu

CASES = [
    # (act, n, m, b).  Splits of 288 tokens, too short for the straight-to-LDS
    # tile: the bounds-checked kernel, last splits of 1, 63 and 225 tokens
    ("bf16", (8, 8, 8), (8, 8, 8), 2049 + 256),
    ("bf16", (8, 8, 8), (8, 8, 8), 2111 + 256),
    ("bf16", (8, 8, 8), (8, 8, 8), 7 * 320 + 1),
    # 12 splits of 320 tokens and one of 161
    ("bf16", (8, 8, 12), (12, 8, 8), 4001),
    # 768 x 768 fp32: 7 splits of 288 tokens and one of 33, of 63
    ("f32", (8, 8, 12), (12, 8, 8), 2049),
    ("f32", (8, 8, 12), (12, 8, 8), 2079),
    # 9 splits of 288 tokens and one of 13, less than a stage
    ("f32", (17, 8, 8), (8, 16, 8), 2605),
    # a last split of one token, and of 127 (63 past a whole stage)
    ("bf16", (8, 8, 12), (12, 8, 8), 12 * 320 + 1),
    ("bf16", (8, 8, 8), (8, 8, 8), 20 * 320 + 127),
    ("f32", (8, 8, 12), (12, 8, 8), 8 * 288 + 1),
    # one split of less than a stage
    ("bf16", (16, 16, 16), (16, 16, 16), 17),
]


@pytest.mark.parametrize("case", CASES, ids=[f"{c[0]}_{c[3]}" for c in CASES])
def test_short_last_stage(case):
    act, n, m, b = case
    print(f"dw tail {case}", flush=True)
    r = (1, 6, 7, 1)
    cores, D, X, dY = _inputs(141, n, m, r, b, act)
    dGr = OT.backward_dense(X, dY, cores, D)[1]
    run = TTMRun(n, m, r, cores, D, b, act, force_order=0)
    dG = run.backward(to_dev(X, act), to_dev(dY, act), want_dx=False)[1]
    errs = [rel_err(to_np(g), ref) for g, ref in zip(dG, dGr)]
    assert max(errs) <= 1e-4, errs
