"""Which kernels a call launches, on the CPU: the calls run their host path in
the library's launch check mode (placeholder pointers, no device memory
touched) and the recorded kernel names say which route was taken.  Both sides
of every line that a route's rule draws."""
import math

import pytest

from paper_2405_14377_amd import comera as C
from tests.launch_sizing_cases import fake

ACT = {"f32": C.F32, "bf16": C.BF16}


def _order(plan, desc):
    for i in range(plan.num_orders):
        info = plan.order_info(i)
        if info["desc"] == desc:
            return i, info["executable"]
    raise AssertionError(desc)


def layer_kernels(n, m, r, act, b, order=-1, want_dx=True, want_dg=True, reuse=True):
    """(forward, backward) kernel names of one layer in launch order, and its
    workspace bytes; order: an index, -1 or the text of order_info."""
    d = len(n)
    if isinstance(order, str):
        order, ok = _order(C.TTMPlan(n, m, r, ACT[act], batch=b), order)
        assert ok, "the order is not executable"
    p = C.TTMPlan(n, m, r, ACT[act], batch=b, force_order=order)
    p.set_reuse_forward(reuse)
    esz = 2 if act == "bf16" else 4
    lib, wsb = C.load(), p.workspace_bytes
    cores = [4 * r[k] * m[k] * n[k] * r[k + 1] for k in range(d)]
    G, dG = (C._ptr_array([fake(x) for x in cores]) for _ in range(2))
    X, dX = (fake(esz * b * math.prod(n)) for _ in range(2))
    Y, dY = (fake(esz * b * math.prod(m)) for _ in range(2))
    ws = fake(wsb)
    out = []
    for call in (lambda: lib.comera_ttm_forward(p.handle, b, X, G, None, Y, ws, wsb, 0),
                 lambda: lib.comera_ttm_backward(p.handle, b, X, dY, G, None, dX if want_dx else None,
                                                 dG if want_dg else None, ws, wsb, 0)):
        C.comera_debug_launch_check(True)
        try:
            assert call() == C.OK
            log = C.comera_debug_launch_log()
        finally:
            C.comera_debug_launch_check(False)
        assert all(x["ok"] for x in log), [x for x in log if not x["ok"]]
        out.append([x["kernel"] for x in log])
    return out[0], out[1], wsb


# ------------------------------------------------------------------ the two-group sweep through one bond
@pytest.mark.parametrize("act,n,m,r", [
    # a folded core of 2^31 entries at its padded rank, below that unpadded
    ("f32", (4, 1048576, 1), (1, 1, 8), (1, 64, 1, 1)),
    ("f32", (4, 1048576, 1), (1, 1, 8), (1, 64, 2, 1)),
    ("bf16", (8, 524288, 1), (1, 1, 256), (1, 64, 40, 1)),
])
def test_one_bond_refuses_cores_past_32_bits(act, n, m, r):
    fwd, bwd, _ = layer_kernels(n, m, r, act, 16, "sweep-lr [0,1][2]")
    assert "tt_build_kernel" not in fwd + bwd


def _tt(ins, outs, rank):
    k, q = len(ins), len(ins) + len(outs)
    desc = "sweep-lr [" + ",".join(map(str, range(k))) + "][" + ",".join(map(str, range(k, q))) + "]"
    return ins + (1,) * len(outs), (1,) * k + outs, (1,) + (rank,) * (q - 1) + (1,), desc


@pytest.mark.parametrize("act,ins,outs,rank,b,own", [
    # rounds of the build: 16 and 17 over modes of 64 and 65 x 8
    ("bf16", (64, 64), (64, 64), 32, 4096, True), ("bf16", (64, 64), (72, 64), 32, 4096, False),
    ("f32", (64, 72), (64, 64), 32, 4096, False), ("bf16", (32, 24), (48, 64), 64, 4096, False),
    ("bf16", (8, 8, 12), (16, 16, 16), 64, 4096, True), ("bf16", (8, 8, 12), (17, 16, 16), 64, 4096, False),
    ("f32", (128,), (128,), 32, 4096, True), ("f32", (768,), (768,), 32, 4096, False),
    # fp32 at a padded rank of 64 over few and many tokens
    ("f32", (8, 8, 12), (16, 16, 12), 33, 63, False), ("f32", (8, 8, 12), (16, 16, 12), 33, 64, True),
    ("f32", (8, 8, 12), (16, 16, 12), 48, 16384, True), ("f32", (8, 8, 12), (16, 16, 12), 48, 16385, False),
    ("f32", (8, 8, 12), (16, 16, 12), 32, 16385, True), ("bf16", (8, 8, 12), (16, 16, 12), 48, 16385, True),
    # rows past 4096 columns
    ("f32", (8, 8, 12), (16, 16, 16), 32, 7, True), ("f32", (8, 8, 12), (16, 16, 16), 48, 4096, True),
    ("f32", (8, 8, 12), (17, 16, 16), 32, 4096, False), ("bf16", (8, 8, 12), (16, 16, 16), 40, 7, True),
    ("bf16", (8, 8, 12), (17, 16, 16), 32, 511, False), ("bf16", (8, 8, 12), (17, 16, 16), 32, 512, True),
    ("bf16", (8, 8, 12), (17, 16, 14), 40, 512, True), ("bf16", (8, 8, 12), (16, 24, 16), 40, 512, False),
])
def test_one_bond_kernels_where_they_are_faster(act, ins, outs, rank, b, own):
    n, m, r, desc = _tt(ins, outs, rank)
    fwd, bwd, _ = layer_kernels(n, m, r, act, b, desc)
    if own:
        assert fwd == ["tt_build_kernel", "tt_pass_kernel"]
        assert bwd[:2] == ["tt_pass_kernel", "tt_meet_kernel"] and bwd[-1] == "tt_grad_kernel"
    else:
        assert not [k for k in fwd + bwd if k.startswith("tt_")]
