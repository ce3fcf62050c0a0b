"""Short calls: selection of a short history in one workgroup (edges of its range, more pooled rows than one pass
holds), append for every element type / head dim, and workspaces sized for another length of the history."""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs, to_numpy, torch_dtype

import parity_util as pu

pytestmark = pytest.mark.gpu


def _desc(w, x):
    return api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, torch_dtype(w.grad_dtype))


# One workgroup per KV head selects where n_past + m * G <= 192 (here m * G = 4, so up to 188 pages), in three groups of 64 pages;
# from 189 on the ordinary kernels do
@pytest.mark.parametrize("dtype,D,P", [("f32", 64, 16), ("bf16", 128, 128), ("bf16", 64, 32)])
@pytest.mark.parametrize("n_past", [1, 63, 64, 65, 127, 128, 129, 187, 188, 189, 192, 193])
def test_selection_of_short_histories(n_past, dtype, D, P):
    w = Workload("short", 4, 2, D, P, 2 * P, (n_past + 2) * P, min(n_past, 9), dtype, "f32", 0.1, extra_phys=2, seed=400 + n_past)
    x = make_inputs(w, "cuda")
    ran = ("select_small", "topk_select") if n_past <= 188 else ("topk_select", "select_small")
    with pu.kernels_ran(ran[:1], absent=ran[1:]):
        sel, cnt, scores = pu.gpu_select(w, x)
    osel, ocnt, oscores = pu.oracle_select(w, pu.host_inputs(x))
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
    assert np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(cnt.cpu().numpy(), ocnt)


# Equal scores on both sides of pages 64 and 128: groups of pages with the same mean, zeros of either sign, ties to the lower page
@pytest.mark.parametrize("n_past", [64, 65, 130, 188])
def test_selection_of_short_histories_with_tied_scores(n_past):
    hkv, D, P, m = 2, 64, 16, 2
    g = torch.Generator(device="cuda").manual_seed(480 + n_past)
    n = n_past + m
    base = torch.randn((4, hkv, D), generator=g, device="cuda")
    base[2], base[3] = 0.0, -0.0
    kbar = base[torch.randint(0, 4, (n,), generator=g, device="cuda")].contiguous()
    q = torch.randn((m * P, 4, D), generator=g, device="cuda").abs() + 0.1
    desc = api.make_desc(q, torch.empty((1, hkv, P, D), device="cuda").expand(n, hkv, P, D), n * P, 0.125)
    desc.pool_page_stride = hkv * P * D
    for top_k in (1, 5, n_past // 3, 64, n_past - 1, n_past, n_past + 4):
        scores = torch.empty((hkv, n_past), dtype=torch.float32, device="cuda")
        with pu.kernels_ran(("select_small",), absent=("topk_select",)):
            sel, cnt = api.page_score_topk_cached(desc, q, kbar, top_k, scores_out=scores)
        osel, ocnt, oscores = orc.page_score_topk_cached(orc.Shape(4, hkv, D, P, m * P, n * P, 0.125), q.cpu().numpy(), kbar.cpu().numpy(), top_k)
        assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
        assert np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(cnt.cpu().numpy(), ocnt), top_k


@pytest.mark.parametrize("n_past", [300, 1500, 9000])
def test_selection_among_close_scores(n_past):
    # distinct scores that share their leading bits: the cut is found after several passes, among few candidates
    hkv, D, C = 2, 64, 32
    g = torch.Generator(device="cuda").manual_seed(430 + n_past)
    n = n_past + 2
    kbar = torch.randn((1, hkv, D), generator=g, device="cuda") * (1 + torch.randperm(n, generator=g, device="cuda")[:, None, None] * 2.0**-22)
    q = torch.randn((C, 4, D), generator=g, device="cuda")
    desc = api.make_desc(q, torch.empty((1, hkv, 16, D), device="cuda").expand(n, hkv, 16, D), n * 16, 0.125)
    desc.pool_page_stride = hkv * 16 * D
    for top_k in (1, 77, n_past // 2):
        scores = torch.empty((hkv, n_past), dtype=torch.float32, device="cuda")
        sel, cnt = api.page_score_topk_cached(desc, q, kbar, top_k, scores_out=scores)
        osel, ocnt, oscores = orc.page_score_topk_cached(orc.Shape(4, hkv, D, 16, C, n * 16, 0.125), q.cpu().numpy(), kbar.cpu().numpy(), top_k)
        assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
        assert np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(cnt.cpu().numpy(), ocnt)


def test_selection_of_a_short_history_with_many_pooled_rows():
    # m * G = 256: the past fits the kernel of one workgroup per KV head, the rows to pool do not
    w = Workload("rows", 32, 1, 128, 16, 16 * 8, 16 * 48, 7, "bf16", "f32", 0.1, seed=420)
    x = make_inputs(w, "cuda")
    with pu.kernels_ran(("qpool_final",), absent=("select_small",)):
        sel, cnt, scores = pu.gpu_select(w, x)
    osel, ocnt, oscores = pu.oracle_select(w, pu.host_inputs(x))
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
    assert np.array_equal(sel.cpu().numpy(), osel)


# Up to 16 rows to pool and 32768 (head, page) pairs the scoring kernel pools them itself, eight rows at a time, 16 or 32 pages per workgroup
@pytest.mark.parametrize("Hq,Hkv,D,m,n_past", [(2, 2, 128, 1, 209), (8, 1, 128, 1, 207), (9, 1, 64, 1, 225), (14, 2, 128, 1, 1023), (28, 4, 64, 2, 223), (8, 1, 64, 2, 32768),
                                               (16, 2, 128, 2, 208), (17, 1, 128, 1, 208), (3, 1, 64, 6, 193), (4, 1, 64, 1, 32769)])
def test_selection_pools_few_rows_where_it_scores(Hq, Hkv, D, m, n_past):
    g = torch.Generator(device="cuda").manual_seed(440 + n_past)
    P, n = 16, n_past + m
    kbar = torch.randn((n, Hkv, D), generator=g, device="cuda")
    q = torch.randn((m * P, Hq, D), generator=g, device="cuda")
    desc = api.make_desc(q, torch.empty((1, Hkv, P, D), device="cuda").expand(n, Hkv, P, D), n * P, 0.125)
    desc.pool_page_stride = Hkv * P * D
    scores = torch.empty((Hkv, n_past), dtype=torch.float32, device="cuda")
    ran = ("page_score_pooled", "qpool_final") if m * Hq // Hkv <= 16 and n_past * Hkv <= 32768 else ("qpool_final", "page_score_pooled")
    with pu.kernels_ran(ran[:1], absent=ran[1:]):
        sel, cnt = api.page_score_topk_cached(desc, q, kbar, 37, scores_out=scores)
    osel, ocnt, oscores = orc.page_score_topk_cached(orc.Shape(Hq, Hkv, D, P, m * P, n * P, 0.125), q.cpu().numpy(), kbar.cpu().numpy(), 37)
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
    assert np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(cnt.cpu().numpy(), ocnt)


# No history: the lists hold the chunk's own pages, whichever kernels would have scored a past.  Pages of 16 and 32 tokens with more
# than 192 rows to pool, and (128 tokens) query sums too large for the built-in scratch.
@pytest.mark.parametrize("Hq,Hkv,D,P,m", [(14, 2, 64, 16, 32), (28, 4, 64, 32, 28), (32, 1, 64, 16, 6), (28, 4, 128, 128, 293)])
def test_selection_without_a_history(Hq, Hkv, D, P, m):
    w = Workload("first", Hq, Hkv, D, P, m * P, m * P, 5, "bf16", "f32", 0.1, seed=410)
    x = make_inputs(w, "cuda", zero_grad_pools=False)
    want = np.broadcast_to(np.concatenate([np.arange(m), -np.ones(5)]), (Hkv, m + 5))
    calls = [lambda *a: api.page_score_topk(*a)]
    if Hq * m * D + Hkv * D <= api.NOALLOC_SCRATCH_BYTES // 4 - 256:
        calls.append(lambda *a: api.page_score_topk_noalloc(*a, torch.full((Hkv, m + 5), 9, dtype=torch.int32, device="cuda"),
                                                            torch.full((Hkv,), 9, dtype=torch.int32, device="cuda")))
    for call in calls:
        sel, cnt = call(_desc(w, x), x["q"], x["k_pool"], x["page_table"], 5)
        assert np.array_equal(sel.cpu().numpy(), want) and (cnt.cpu().numpy() == m).all()


# Rows to pool around what the kernel that pools them holds at once (1024 rows of 16 dims), and past it
@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("m", [62, 63, 64, 65, 100, 129])
def test_selection_pools_more_rows_than_fit_at_once(m, dtype):
    w = Workload("rows", 16, 1, 64, 16, 16 * m, 16 * (m + 30), 7, dtype, "f32", 0.1, seed=421)
    x = make_inputs(w, "cuda")
    sel, cnt, scores = pu.gpu_select(w, x)
    osel, ocnt, oscores = pu.oracle_select(w, pu.host_inputs(x))
    assert np.array_equal(scores.cpu().numpy().view(np.uint32), oscores.view(np.uint32))
    assert np.array_equal(sel.cpu().numpy(), osel)


# The scoring workspace needs no alignment beyond that of its floats
@pytest.mark.parametrize("n_past,P,m", [(20, 64, 2), (300, 64, 2), (300, 16, 40), (700, 16, 2)])
def test_selection_in_a_workspace_at_any_float(n_past, P, m):
    w = Workload("offset", 4, 2, 64, P, m * P, (n_past + m) * P, 9, "f32", "f32", 0.1, seed=425)
    x = make_inputs(w, "cuda", zero_grad_pools=False)
    desc = _desc(w, x)
    osel, ocnt, _ = pu.oracle_select(w, pu.host_inputs(x))
    kbar = torch.zeros((w.n, w.Hkv, w.D), dtype=torch.float32, device="cuda")
    api.page_means(desc, x["k_pool"], x["page_table"], 0, w.n, kbar)
    need = api.workspace_bytes(desc, w.top_k, api.OP_SCORE_TOPK)
    big = torch.empty(need + 16, dtype=torch.uint8, device="cuda")
    for off in (0, 4, 8, 12):
        ws = big[off:off + need]
        for sel, cnt in (api.page_score_topk(desc, x["q"], x["k_pool"], x["page_table"], w.top_k, workspace=ws),
                         api.page_score_topk_cached(desc, x["q"], kbar, w.top_k, workspace=ws)):
            assert np.array_equal(sel.cpu().numpy(), osel) and np.array_equal(cnt.cpu().numpy(), ocnt)


@pytest.mark.parametrize("with_means", [True, False])
@pytest.mark.parametrize("dtype,D,P", [("f32", 128, 128), ("f32", 64, 16), ("bf16", 64, 128), ("bf16", 128, 16)])
def test_append_for_every_tile(dtype, D, P, with_means):
    w = Workload("append", 3, 3, D, P, 3 * P, 8 * P, None, dtype, "f32", 0.1, extra_phys=1, seed=430)
    x = make_inputs(w, "cuda")
    sh, dt = pu.shape_of(w), x["k_pool"].dtype
    gen = torch.Generator(device="cpu").manual_seed(431)
    kc, vc = (torch.randn((w.C, w.Hkv, w.D), generator=gen).to(dt).cuda() for _ in range(2))
    cache = torch.full((sh.n, w.Hkv, w.D), 7.0, dtype=torch.float32, device="cuda")
    ok, ov, oc = orc.kv_append(sh, to_numpy(kc), to_numpy(vc), to_numpy(x["page_table"]), to_numpy(x["k_pool"]), to_numpy(x["v_pool"]), cache.cpu().numpy())
    api.kv_append(_desc(w, x), kc, vc, x["page_table"], x["k_pool"], x["v_pool"], cache if with_means else None)
    torch.cuda.synchronize()
    assert np.array_equal(to_numpy(x["k_pool"]), ok) and np.array_equal(to_numpy(x["v_pool"]), ov)
    if with_means:
        assert np.array_equal(cache.cpu().numpy().view(np.uint32), oc.view(np.uint32))


@pytest.mark.parametrize("dtype,P,top_k", [("bf16", 128, None), ("bf16", 128, 4), ("f32", 64, None)])
def test_a_workspace_of_the_longest_history_serves_the_shorter_ones(dtype, P, top_k):
    last = Workload("grow", 6, 2, 128, P, 2 * P, 26 * P, top_k, dtype, "f32", 0.0884, seed=440)
    x = make_inputs(last, "cuda")
    hx = pu.host_inputs(x)
    lk = -1 if top_k is None else top_k
    ws = {op: torch.empty(api.workspace_bytes(_desc(last, x), k, op), dtype=torch.uint8, device="cuda")
          for op, k in ((api.OP_SCORE_TOPK, top_k or 0), (api.OP_ATTN_FWD, lk), (api.OP_ATTN_BWD, lk))}
    for n in (2, 3, 7, 13, 26):
        w = last.with_(N=n * P)
        desc = _desc(w, x)
        sel = cnt = osel = ocnt = None
        if top_k is not None:
            sel, cnt = api.page_score_topk(desc, x["q"], x["k_pool"], x["page_table"], top_k, workspace=ws[api.OP_SCORE_TOPK])
            osel, ocnt, _ = orc.page_score_topk(pu.shape_of(w), hx["q"], hx["k_pool"], hx["page_table"], top_k)
            assert np.array_equal(sel.cpu().numpy(), osel)
        x["dk_pool"].zero_()
        x["dv_pool"].zero_()
        o, lse = api.paged_attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], sel, cnt, workspace=ws[api.OP_ATTN_FWD])
        dq = api.paged_attn_bwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], sel, cnt,
                                workspace=ws[api.OP_ATTN_BWD])
        ref = pu.oracle_fwd_bwd(w, hx, osel, ocnt)
        for name, got, want in (("O", o, ref["o"]), ("dQ", dq, ref["dq"]), ("dK", x["dk_pool"], ref["dk_pool"]), ("dV", x["dv_pool"], ref["dv_pool"])):
            pu.check(name, pu.f32(got), want, dtype)


@pytest.mark.parametrize("dtype,D,P", [("bf16", 128, 128), ("bf16", 64, 32), ("f32", 64, 16)])
def test_dq_may_be_written_over_o(dtype, D, P):
    # short calls, whose dQ and dK / dV otherwise run side by side, both reading O; the same sums in another split
    w = Workload("over", 4, 2, D, P, 2 * P, 9 * P, None, dtype, "f32", D ** -0.5, seed=450)
    x = make_inputs(w, "cuda")
    desc = _desc(w, x)
    args = (x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(desc, *args)
    x["dk_pool"].zero_()
    x["dv_pool"].zero_()
    dq = api.paged_attn_bwd(desc, *args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], d_q=o)
    assert dq.data_ptr() == o.data_ptr()
    ref = pu.oracle_fwd_bwd(w, pu.host_inputs(x), None, None)
    for name, got, want in (("dQ", dq, ref["dq"]), ("dK", x["dk_pool"], ref["dk_pool"]), ("dV", x["dv_pool"], ref["dv_pool"])):
        pu.check(name, pu.f32(got), want, dtype)


# dQ over O one row further on, one head further on, and beside it in the same rows
@pytest.mark.parametrize("how", ["row", "head", "beside"])
@pytest.mark.parametrize("dtype,D,P,n,Hq,m", [("bf16", 128, 128, 9, 4, 2), ("bf16", 64, 32, 9, 4, 2), ("f32", 64, 16, 9, 4, 2), ("f32", 128, 16, 40, 32, 24),
                                              ("bf16", 64, 16, 80, 28, 40)])
def test_dq_may_overlap_o(dtype, D, P, n, Hq, m, how):
    w = Workload("overlap", Hq, 2, D, P, m * P, (n + m) * P, None, dtype, "f32", D ** -0.5, seed=460)
    x = make_inputs(w, "cuda")
    big = torch.empty((w.C + 1, Hq, 2 * D if how == "beside" else D), dtype=x["q"].dtype, device="cuda")
    flat, size = big.view(-1), w.C * Hq * D
    if how == "beside":
        o, dq = big[:-1, :, :D], big[:-1, :, D:]
        for k in ("q", "d_o"):
            x[k] = torch.empty_like(big)[:-1, :, :D].copy_(x[k])
    else:
        at = Hq * D if how == "row" else D
        o, dq = flat[:size].view(x["q"].shape), flat[at:at + size].view(x["q"].shape)
    desc = _desc(w, x)
    args = (x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(desc, *args, o=o)
    api.paged_attn_bwd(desc, *args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], d_q=dq)
    ref = pu.oracle_fwd_bwd(w, pu.host_inputs(x), None, None)
    for name, got, want in (("dQ", dq, ref["dq"]), ("dK", x["dk_pool"], ref["dk_pool"]), ("dV", x["dv_pool"], ref["dv_pool"])):
        pu.check(name, pu.f32(got), want, dtype)


@pytest.mark.parametrize("dtype,D,P", [("bf16", 128, 128), ("f32", 64, 16)])
def test_lists_may_be_a_view_that_ends_before_its_stride(dtype, D, P):
    w = Workload("view", 4, 2, D, P, 2 * P, 9 * P, 3, dtype, "f32", D ** -0.5, seed=470)
    x = make_inputs(w, "cuda")
    desc = _desc(w, x)
    sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
    view = torch.full((w.Hkv, 9), -7, dtype=torch.int32, device="cuda")[:, 4:].copy_(sel)
    args = (x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(desc, *args, view, cnt)
    dq = api.paged_attn_bwd(desc, *args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], view, cnt)
    ref = pu.oracle_fwd_bwd(w, pu.host_inputs(x), sel.cpu().numpy(), cnt.cpu().numpy())
    for name, got, want in (("O", o, ref["o"]), ("dQ", dq, ref["dq"]), ("dK", x["dk_pool"], ref["dk_pool"]), ("dV", x["dv_pool"], ref["dv_pool"])):
        pu.check(name, pu.f32(got), want, dtype)


# Logits that rise by `rise` binary orders per 32 keys: references that stay where they are (up to 2^8 above), move now and then, and move in every tile.  fp32: a logit
# of L is off by 2^-24 L a few times over, and so is the logarithm of what it weighs; bf16: O is rounded to 8 bits.
@pytest.mark.parametrize("dtype,D,P,C,n", [("f32", 64, 16, 64, 12), ("f32", 128, 128, 512, 20), ("bf16", 64, 16, 64, 24), ("bf16", 128, 64, 128, 9)])
@pytest.mark.parametrize("rise", [0.4, 3.0, 9.0])
def test_forward_of_rising_logits(dtype, D, P, C, n, rise):
    w = Workload("rising", 28 if C == 512 else 2, 4 if C == 512 else 1, D, P, C, P * n, None, dtype, "f32", 1.0, seed=700 + n)
    x = make_inputs(w, "cuda")
    q, kp, vp, table = x["q"], x["k_pool"], x["v_pool"], x["page_table"].long()
    t = torch.arange(w.N, device="cuda").reshape(n, 1, P, 1)
    kp[table] = (kp[table].double() * 0.02 + t * (rise * math.log(2) / 32 / D)).to(kp.dtype)
    q.copy_(1 + 0.05 * q.float())
    o, lse = api.paged_attn_fwd(api.make_desc(q, kp, w.N, 1.0), q, kp, vp, table.int(), None, None)
    K, V = (p[table].double().transpose(0, 1).reshape(w.Hkv, w.N, D).repeat_interleave(w.G, 0) for p in (kp, vp))
    s = torch.matmul(q.double().transpose(0, 1), K.transpose(1, 2).contiguous())
    s = s.masked_fill(torch.arange(w.N, device="cuda") > torch.arange(w.N - C, w.N, device="cuda")[:, None], -math.inf)
    want, top = torch.matmul(torch.softmax(s, 2), V).transpose(0, 1), s[s > -math.inf].abs().max().item()
    line = 4 * 2.0**-24 * max(top, 4.0) if dtype == "f32" else 2.0**-8
    assert ((o.double() - want).norm() / want.norm()).item() < line
    assert (lse.double() - torch.logsumexp(s, 2)).abs().max().item() < 4 * 2.0**-24 * max(top, 8.0)
    if dtype == "f32":   # the same average of values whose unnormalised sum is out of range
        vp.fill_(2.5e38)
        o, _ = api.paged_attn_fwd(api.make_desc(q, kp, w.N, 1.0), q, kp, vp, table.int(), None, None)
        assert (o.double() / 2.5e38 - 1).abs().max().item() < 4 * 2.0**-24 * max(top, 4.0) + w.N * 2.0**-24
