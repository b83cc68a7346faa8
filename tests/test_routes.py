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


def test_one_bond_kernels_of_the_gpu_cases():
    """The GPU parity cases reach the kernels that they are for."""
    from tests.test_gpu_bottleneck import SHAPES, _layout
    cases = [(ins, outs, ranks, b) for _, ins, outs, ranks, b in SHAPES]
    cases += [((8, 4), (4, 16), (6, 10, 6), b) for b in (8200, 16400)]
    cases += [((4, 3, 4), (4, 4, 3), (4, 12, 40, 12, 4), 200), ((4, 4, 6), (6, 4, 4), (5, 6, 7, 6, 5), 90)]
    cases += [((4, 6), (8, 4), x, 72) for x in ((3, 1, 2), (6, 30, 7), (6, 33, 7))]
    for ins, outs, ranks, b in cases:
        n, m, r = _layout(ins, outs, ranks)
        desc = _tt(ins, outs, 1)[3]
        for act in ("f32", "bf16"):
            fwd, bwd, _ = layer_kernels(n, m, r, act, b, desc)
            assert fwd == ["tt_build_kernel", "tt_pass_kernel"], (ins, outs, ranks, b, act)
            assert "tt_meet_kernel" in bwd and "tt_grad_kernel" in bwd


# ------------------------------------------------------------------ products of few rows
_F = {512: (8, 8, 8), 768: (8, 8, 12), 1000: (10, 10, 10), 1024: (8, 8, 16), 1280: (8, 10, 16), 1536: (8, 12, 16),
      2048: (8, 16, 16), 3072: (16, 16, 12), 4096: (16, 16, 16), 8192: (16, 16, 32), 16384: (32, 16, 32),
      496: (8, 2, 31), 770: (7, 10, 11), 792: (9, 11, 8), 680: (5, 8, 17)}


@pytest.mark.parametrize("act,K,N,b,own", [
    ("bf16", 768, 3072, 1, True), ("bf16", 4096, 512, 16, True), ("bf16", 8192, 512, 16, False),
    ("bf16", 512, 8192, 16, True), ("bf16", 512, 16384, 16, False), ("bf16", 768, 496, 16, False),
    ("bf16", 1024, 768, 32, True), ("bf16", 1280, 512, 17, False), ("bf16", 2048, 4096, 32, True),
    ("bf16", 3072, 4096, 32, False), ("bf16", 2048, 8192, 32, False), ("bf16", 768, 3072, 33, True),
    ("bf16", 768, 512, 64, True), ("bf16", 1024, 512, 64, False), ("bf16", 1536, 4096, 64, True),
    ("bf16", 2048, 4096, 64, False), ("bf16", 4096, 512, 64, False), ("bf16", 768, 3072, 65, False),
    ("bf16", 770, 768, 7, False), ("bf16", 680, 792, 33, True),
    ("f32", 16384, 512, 16, True), ("f32", 4096, 4096, 16, True), ("f32", 1024, 512, 32, True),
    ("f32", 1280, 512, 32, False), ("f32", 1280, 2048, 32, True), ("f32", 3072, 768, 32, True),
    ("f32", 4096, 512, 32, False), ("f32", 768, 3072, 64, True), ("f32", 768, 512, 64, False),
    ("f32", 1000, 3072, 64, False), ("f32", 768, 16384, 64, False), ("f32", 768, 3072, 65, False),
])
def test_few_rows_kernel_where_it_is_faster(act, K, N, b, own):
    fwd, _, _ = layer_kernels(_F[K], _F[N], (1, 4, 4, 1), act, b, 0)
    assert ("gemm_skinny_kernel" in fwd) == own


def test_few_rows_kernel_of_the_gpu_cases():
    """The GPU parity cases reach every form of the kernel: 16, 32 and 64 rows
    in both dtypes, K and N that are no whole number of steps or tiles."""
    from tests.test_gpu_skinny import SHAPES
    own = {(act, b, i) for act in ACT for b in (1, 7, 16, 17, 32, 33, 64, 65) for i, (n, m) in enumerate(SHAPES)
           if "gemm_skinny_kernel" in layer_kernels(n, m, (1, 6, 7, 1), act, b, 0)[0]}
    assert {(act, b) for act, b, _ in own} == {(act, b) for act in ACT for b in (1, 7, 16, 17, 32, 33, 64)}
    assert {i for _, b, i in own if b <= 16} == {0, 1, 2} and {i for a, b, i in own if a == "bf16" and b > 32} == {0, 1}


def test_few_rows_dx_keeps_the_splits_of_the_plan():
    """fp32 dX over N_out >= 1024 is split over K by the plan and stays so;
    bf16 and narrower fp32 layers take the few-rows kernel."""
    assert "gemm_skinny_kernel" not in layer_kernels(_F[768], _F[3072], (1, 4, 4, 1), "f32", 7, 0, want_dg=False)[1]
    assert "gemm_skinny_kernel" in layer_kernels(_F[768], _F[3072], (1, 4, 4, 1), "bf16", 7, 0, want_dg=False)[1]
    assert "gemm_skinny_kernel" in layer_kernels(_F[680], _F[792], (1, 4, 4, 1), "f32", 7, 0, want_dg=False)[1]


# ------------------------------------------------------------------ dW over a token count that ends within a stage
@pytest.mark.parametrize("act,n,m,b,own", [
    ("f32", (16, 16, 12), (16, 16, 12), 199, False), ("f32", (16, 16, 12), (16, 16, 12), 201, True),
    ("f32", (16, 16, 16), (16, 16, 16), 17, False), ("f32", (8, 8, 12), (12, 8, 8), 2049, True),
    ("bf16", (8, 12, 16), (16, 16, 12), 299, False), ("bf16", (8, 12, 16), (16, 16, 12), 301, True),
    ("bf16", (16, 16, 16), (16, 16, 16), 17, True), ("bf16", (8, 8, 12), (12, 8, 8), 16001, True),
    # a last output mode that is no whole number of 16-byte pieces
    ("bf16", (12, 14, 10), (12, 14, 10), 3333, False), ("bf16", (12, 14, 10), (12, 14, 10), 4001, True),
    ("bf16", (16, 16, 12), (12, 10, 15), 2001, False), ("bf16", (16, 16, 12), (12, 10, 15), 3333, True),
])
def test_dw_tail_where_it_is_faster(act, n, m, b, own):
    _, bwd, _ = layer_kernels(n, m, (1, 4, 4, 1), act, b, 0, want_dx=False)
    assert any(k.endswith("<tail>") for k in bwd) == own, bwd


def test_dw_tail_of_the_gpu_cases():
    """The GPU parity cases reach the kernel that they are for."""
    from tests.test_gpu_dw_tail import CASES
    own = []
    for act, n, m, b in CASES:
        _, bwd, _ = layer_kernels(n, m, (1, 6, 7, 1), act, b, 0, want_dx=False)
        if any(k.endswith("<tail>") for k in bwd):
            own.append((act, b))
    assert own == [("bf16", 4001), ("f32", 2049), ("f32", 2079), ("f32", 2605), ("bf16", 3841), ("bf16", 6527),
                   ("f32", 2305), ("bf16", 17)]


# ------------------------------------------------------------------ FP8 quantiser
@pytest.mark.parametrize("act,rows,cols,name,nb", [
    ("bf16", 64, 64, "amax_vec_kernel", 1), ("bf16", 16384, 1024, "amax_vec_kernel", 512),
    ("bf16", 8192, 1024, "amax_vec_kernel", 256), ("bf16", 8192, 4096, "amax_vec_kernel", 512),
    ("bf16", 8192, 4104, "amax_vec_kernel<wide>", 512), ("f32", 16384, 1024, "amax_vec_kernel", 512),
    ("f32", 40000, 4096, "amax_vec_kernel<wide>", 512),
])
def test_maximum_pass_leaves_no_workgroup_without_loads(act, rows, cols, name, nb):
    C.comera_debug_launch_check(True)
    try:
        assert C.load().comera_fp8_quantize(fake(4 * rows * cols), ACT[act], rows, cols, fake(rows * cols), cols, None,
                                            0, fake(4), fake(4096), C.FP8_QUANTIZE_WS_BYTES, 0) == C.OK
        log = C.comera_debug_launch_log()
    finally:
        C.comera_debug_launch_check(False)
    assert (log[0]["kernel"], log[0]["grid"][0]) == (name, nb)
    chunks = rows * cols // (8 if act == "bf16" else 4)
    assert (nb - 1) * 1024 * (8 if "wide" in name else 4) < chunks


# ------------------------------------------------------------------ embedding
@pytest.mark.parametrize("v,n,rows_ahead,da_ahead", [
    ((30, 31, 33), 4095, False, False), ((30, 31, 33), 4096, True, False), ((30, 31, 33), 12 * 930, True, True),
    ((30, 31, 24), 12 * 930, True, True), ((30, 31, 23), 12 * 930, True, False), ((30, 31, 33), 12 * 930 - 1, True, False),
    ((4, 5, 32), 240, False, True),
])
def test_embedding_loads_ahead(v, n, rows_ahead, da_ahead):
    e, r = (8, 8, 12), (1, 30, 30, 1)
    s = C.tt_embed_shape(v, e, r)
    wsb = C.comera_tt_embed_workspace_bytes(s, n)
    G, dG = (C._ptr_array([fake(4 * r[k] * v[k] * e[k] * r[k + 1]) for k in range(3)]) for _ in range(2))
    ids, Y, dY, ws, lib = fake(8 * n), fake(4 * n * 768), fake(4 * n * 768), fake(wsb), C.load()
    C.comera_debug_launch_check(True)
    try:
        assert lib.comera_tt_embed_forward(s, ids, n, G, None, Y, ws, wsb, None, 0) == C.OK
        assert lib.comera_tt_embed_backward(s, ids, n, dY, G, None, dG, 1, ws, wsb, None, 0) == C.OK
        names = [x["kernel"] for x in C.comera_debug_launch_log()]
    finally:
        C.comera_debug_launch_check(False)
    assert ("embed_rows_mfma_kernel<ahead>" in names, "embed_rows_mfma_kernel" in names) == (rows_ahead, not rows_ahead)
    assert ("embed_dapre_mfma_kernel<ahead>" in names, "embed_dapre_mfma_kernel" in names) == (da_ahead, not da_ahead)


def test_embedding_loads_ahead_in_the_gpu_cases():
    """The GPU parity cases take the rows' loads ahead in every form, and both
    forms of dA."""
    from tests.test_gpu_embed import AHEAD
    assert {math.prod(e[:-1]) // 16 for _, e, _ in AHEAD} == set(range(1, 9))
    assert {(r[-2] + 3) // 4 > 4 for _, _, r in AHEAD} == {True, False}
    assert {v[-1] >= 24 for v, _, _ in AHEAD} == {True, False}
    assert all(4099 >= 12 * math.prod(v[:-1]) for v, _, _ in AHEAD)


# ------------------------------------------------------------------ outputs over inputs
def _backward_log(n, m, r, b, order, over):
    p = C.TTMPlan(n, m, r, C.F32, batch=b, force_order=order)
    X, dY, other = (fake(4 * b * math.prod(n)) for _ in range(3))
    G, dG = (C._ptr_array([fake(4 * r[k] * m[k] * n[k] * r[k + 1]) for k in range(len(n))]) for _ in range(2))
    C.comera_debug_launch_check(True)
    try:
        assert C.load().comera_ttm_backward(p.handle, b, X, dY, G, None, {"X": X, "dY": dY, None: other}[over], dG,
                                            fake(p.workspace_bytes), p.workspace_bytes, 0) == C.OK
        return C.comera_debug_launch_log()
    finally:
        C.comera_debug_launch_check(False)


def test_fused_sweep_backward_in_place_keeps_one_workgroup_per_token_group():
    n, m, r = (8, 8, 12), (12, 8, 8), (1, 8, 8, 1)
    rows = {o: [x["grid"][1] for x in _backward_log(n, m, r, 32, 7, o) if "chain_bwd" in x["kernel"]]
            for o in (None, "X", "dY")}
    assert rows == {None: [4], "X": [1], "dY": [1]}


def test_forward_in_place_keeps_split_k():
    n, m, r, b = (8, 8, 12), (12, 8, 8), (1, 6, 7, 1), 16
    p = C.TTMPlan(n, m, r, C.BF16, batch=b, force_order=0)
    X, Y = fake(2 * b * 768), fake(2 * b * 768)
    G = C._ptr_array([fake(4 * r[k] * m[k] * n[k] * r[k + 1]) for k in range(3)])
    names = {}
    for key, out in (("apart", Y), ("in place", X)):
        C.comera_debug_launch_check(True)
        try:
            assert C.load().comera_ttm_forward(p.handle, b, X, G, None, out, fake(p.workspace_bytes),
                                               p.workspace_bytes, 0) == C.OK
            names[key] = [x["kernel"] for x in C.comera_debug_launch_log()]
        finally:
            C.comera_debug_launch_check(False)
    assert "gemm_skinny_kernel" in names["apart"] and "gemm_skinny_kernel" not in names["in place"]
    assert any("sum_splits" in k for k in names["in place"])
