"""Values at the ends of what the kernels of fp32 tensors, head dim 64 and pages of 16 to 64 tokens take: sums that
cancel (every bit of a probability counts), infinities and NaN in tokens that a row does not see, scores far below zero."""
import math

import numpy as np
import pytest
import torch

import oracle as orc
from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs, torch_dtype

import parity_util as pu
from test_gpu_qp_attention import rand_qp_lists

pytestmark = pytest.mark.gpu


def _bf(x):
    return x.to(torch.bfloat16).double()


def _cancelling(weight, count, seed):
    """bf16 values [len(weight)][count] whose sums with `weight` are about 2^-15 of their terms: all random but two, of which the
    first cancels the sum of the others to its own rounding and the second cancels 31/32 of what that leaves."""
    g = torch.Generator().manual_seed(seed)
    v = _bf(torch.randn((len(weight), count), generator=g))
    a, b = torch.topk(weight.abs(), 2).indices.tolist()
    v[a] = v[b] = 0
    v[a] = _bf(-(weight @ v) / weight[a])
    v[b] = _bf(-(weight @ v) / weight[b] * (1 - 1 / 32))
    return v


def _rel(got, want):
    return float((got.double().cpu() - want).norm() / want.norm())


# Probabilities and dS of bf16 tensors are held in 32 bits where a shape has no kernels of its own, also where the result is
# stored in bf16.  Bound: weights off by 2^-24 of themselves, rounding of the exponent included by a few times that, change such a
# sum by 2^-9 to 2^-7, its storage by 2^-9; weights of 17 bits by 3 to 11 %.  2^-6 lies between.
@pytest.mark.parametrize("D,P", [(64, 16), (128, 32), (64, 128)])
def test_cancelling_sums_over_keys(D, P):
    # all rows alike, local keys out of reach: O over dims where dO is 0, dQ over dims where Q is 0
    A, m, n_past = D // 2, 2, 256 // P
    w = Workload("cancel", 4, 2, D, P, m * P, (n_past + m) * P, None, "bf16", "bf16", D ** -0.5, seed=90)
    x = {k: v.cpu() if isinstance(v, torch.Tensor) else v for k, v in make_inputs(w, "cpu").items()}
    x["q"][:] = x["q"][0, 0]
    x["d_o"][:] = x["d_o"][0, 0]
    x["q"][..., A:] = 0
    x["d_o"][..., A:] = 0
    pt = x["page_table"].long()
    past, local = pt[:n_past], pt[n_past:w.n]
    x["k_pool"][..., A:] = 0
    x["k_pool"][local] = -30 * x["q"][0, 0]
    x["v_pool"][local] = 0
    q, do = x["q"][0, 0].double(), x["d_o"][0, 0].double()
    want_o, weights = [], []
    for g in range(w.Hkv):
        k = x["k_pool"][past, g].reshape(-1, D).double()
        s = k @ q * w.sm_scale
        x["v_pool"][past, g, :, A:] = _cancelling(torch.exp(s - s.max()), D - A, 91 + g).reshape(n_past, P, D - A).bfloat16()
        want_o.append(torch.softmax(s, 0) @ x["v_pool"][past, g, :, A:].reshape(-1, D - A).double())
        weights.append(s)
    dev = {k: v.cuda() if isinstance(v, torch.Tensor) else v for k, v in x.items()}
    desc = api.make_desc(dev["q"], dev["k_pool"], w.N, w.sm_scale, torch.bfloat16)
    o, lse = api.paged_attn_fwd(desc, dev["q"], dev["k_pool"], dev["v_pool"], dev["page_table"])
    for g in range(w.Hkv):
        assert _rel(o[:, 2 * g:2 * g + 2, A:], want_o[g].expand(w.C, 2, D - A)) <= 2.0**-6, g
    # the backward on the O and LSE that the forward gave; K may hold anything where Q is 0
    want_dq = []
    for g in range(w.Hkv):
        p = torch.exp(weights[g] - lse[2 * g, 0].double().cpu())
        ds = p * (x["v_pool"][past, g].reshape(-1, D).double() @ do - do @ o[0, 2 * g].double().cpu())
        dev["k_pool"][past.cuda(), g, :, A:] = _cancelling(ds, D - A, 95 + g).reshape(n_past, P, D - A).bfloat16().cuda()
        want_dq.append(ds @ dev["k_pool"][past.cuda(), g, :, A:].reshape(-1, D - A).double().cpu() * w.sm_scale)
    dq = api.paged_attn_bwd(desc, dev["q"], dev["k_pool"], dev["v_pool"], dev["page_table"], o, lse, dev["d_o"], dev["dk_pool"], dev["dv_pool"])
    for g in range(w.Hkv):
        assert _rel(dq[:, 2 * g:2 * g + 2, A:], want_dq[g].expand(w.C, 2, D - A)) <= 2.0**-6, g


@pytest.mark.parametrize("grad_dtype", ["bf16", "f32"])
@pytest.mark.parametrize("D,P", [(64, 16), (128, 32), (64, 128)])
def test_cancelling_sums_over_rows(D, P, grad_dtype):
    # all past keys alike: dV over dims where V is 0, dK over dims where K is 0 (Q and dO may hold anything there)
    A, m, n_past = D // 2, 2, 3
    w = Workload("cancel", 4, 2, D, P, m * P, (n_past + m) * P, None, "bf16", grad_dtype, D ** -0.5, seed=100)
    x = make_inputs(w, "cpu")
    pt = x["page_table"].long()
    past = pt[:n_past]
    for name in ("k_pool", "v_pool"):
        x[name][past] = x[name][past[0], 0, 0].clone()
        x[name][..., A:] = 0
    x["q"][..., A:] = 0
    x["d_o"][..., A:] = 0
    dev = {k: v.cuda() if isinstance(v, torch.Tensor) else v for k, v in x.items()}
    desc = api.make_desc(dev["q"], dev["k_pool"], w.N, w.sm_scale, torch_dtype(grad_dtype))
    o, lse = api.paged_attn_fwd(desc, dev["q"], dev["k_pool"], dev["v_pool"], dev["page_table"])
    k, v = (x[name][past[0], 0, 0].double() for name in ("k_pool", "v_pool"))
    want = []
    for g in range(w.Hkv):
        hs = slice(2 * g, 2 * g + 2)
        p = torch.exp(x["q"][:, hs].double() @ k * w.sm_scale - lse[hs].T.double().cpu())
        ds = p * (x["d_o"][:, hs].double() @ v - (x["d_o"][:, hs].double() * o[:, hs].double().cpu()).sum(-1))
        for name, wt in (("d_o", p), ("q", ds)):
            free = _cancelling(wt.reshape(-1), D - A, 101 + g).reshape(w.C, 2, D - A)
            dev[name][:, hs, A:] = free.bfloat16().cuda()
            want.append((wt.reshape(-1) @ free.reshape(-1, D - A)) * (w.sm_scale if name == "q" else 1.0))
    api.paged_attn_bwd(desc, dev["q"], dev["k_pool"], dev["v_pool"], dev["page_table"], o, lse, dev["d_o"], dev["dk_pool"], dev["dv_pool"])
    for g in range(w.Hkv):
        for pool, ref in (("dv_pool", want[2 * g]), ("dk_pool", want[2 * g + 1])):
            got = dev[pool][past.cuda(), g, :, A:]
            assert _rel(got, ref.expand(n_past, P, D - A)) <= 2.0**-6, (pool, g)


# Probabilities of bf16 pages of 128 are bf16 relative to a running maximum per 32 keys, so the largest key of every 32 up to there
# counts in full: two keys that are each the largest of their 32 give LSE to the last bits (2^-22 of values below 2;
# 2e-4 and more if one of them is rounded to bf16).
@pytest.mark.parametrize("at", [(0, 32), (31, 63), (5, 127), (64, 100)])
@pytest.mark.parametrize("n_past", [1, 5, 33])
def test_the_largest_of_32_keys_is_not_rounded(n_past, at):
    w = Workload("peaks", 4, 2, 128, 128, 128, (n_past + 1) * 128, None, "bf16", "f32", 1.0, seed=105)
    x = make_inputs(w, "cuda")
    x["q"].zero_()
    x["q"][..., 0] = 1
    x["k_pool"][..., 0] = -60
    first = x["page_table"][0].long()
    for t, s in zip(at, (0.0, 1.0)):
        x["k_pool"][first, :, t, 0] = s
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    o, lse = api.paged_attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    assert float((lse.double() - math.log(1 + math.e)).abs().max()) <= 5e-7
    v = x["v_pool"][first].double()
    want = (v[:, at[0]] + math.e * v[:, at[1]]) / (1 + math.e)
    assert float((o.double() - want.repeat_interleave(2, 0)).abs().max()) <= 2.0**-8 * float(want.abs().max())


# Rows and keys split over workgroups or not, several lists, tiles that hold many pages or part of one.
UNSEEN = [
    Workload("f32_split", 14, 2, 64, 16, 48, 16 * 37, 5, "f32", "f32", 0.125, seed=110),
    Workload("bf16_split", 14, 2, 64, 16, 48, 16 * 37, 5, "bf16", "f32", 0.125, seed=111),
    Workload("f32_d128", 6, 3, 128, 128, 256, 128 * 4, None, "f32", "bf16", 0.088, seed=112),
    Workload("bf16_p32", 5, 1, 128, 32, 160, 32 * 23, None, "bf16", "bf16", 0.088, seed=113),
    Workload("f32_rows_unsplit", 32, 32, 64, 64, 1152, 64 * 20, 1, "f32", "f32", 0.125, seed=114),
    Workload("bf16_rows_unsplit", 32, 32, 64, 32, 1152, 32 * 41, 3, "bf16", "f32", 0.125, seed=115),
    Workload("f32_keys_unsplit", 8, 4, 128, 16, 32, 16 * 1100, None, "f32", "f32", 0.088, seed=116),
    # one list per query page, pages held by more lists than a unit of keys takes
    Workload("qp_f32", 4, 2, 64, 16, 16 * 12, 16 * 30, None, "f32", "f32", 0.125, seed=117),
    Workload("qp_bf16_p64", 6, 2, 128, 64, 64 * 11, 64 * 20, None, "bf16", "f32", 0.088, seed=118),
]


def _same_where_finite(name, got, want, dtype):
    """Finite where the oracle is, and within the tolerance there; not finite where the oracle is not."""
    got, want = np.asarray(got, np.float64), np.asarray(want, np.float64)
    ok = np.isfinite(want)
    assert np.array_equal(np.isfinite(got), ok), (name, int((np.isfinite(got) != ok).sum()), got.size)
    pu.check(name, got[ok], want[ok], dtype)


@pytest.mark.parametrize("what", ["v_nan", "v_inf", "k_nan", "do_nan", "q_inf"])
@pytest.mark.parametrize("w", UNSEEN, ids=lambda w: w.name)
def test_values_that_are_not_finite_stay_with_those_who_see_them(w, what):
    x = make_inputs(w, "cuda")
    sel = cnt = osel = ocnt = None
    if w.top_k is not None:
        sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
        osel, ocnt = sel.cpu().numpy(), cnt.cpu().numpy()
    if w.name.startswith("qp_"):
        osel, ocnt = rand_qp_lists(w, 5, w.seed, popular=3)
        sel, cnt = torch.as_tensor(osel, device="cuda"), torch.as_tensor(ocnt, device="cuda")
    attn_fwd, attn_bwd = (api.paged_attn_fwd_qp, api.paged_attn_bwd_qp) if w.name.startswith("qp_") else (api.paged_attn_fwd, api.paged_attn_bwd)
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, torch_dtype(w.grad_dtype))
    fwd = lambda: attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], sel, cnt)
    bad = math.inf if what.endswith("inf") else math.nan
    sh = pu.shape_of(w)
    if what[0] in "kv":   # a token in the middle of the chunk's last page: the rows before it do not see it
        x[what[0] + "_pool"][x["page_table"][w.n - 1].long(), :, w.P // 2 + 3, 3] = bad
        o, lse = fwd()
    else:                 # rows of the chunk's first page: keys after them are not seen by them
        o, lse = fwd()
        x["q" if what[0] == "q" else "d_o"][w.P // 2, :, 3] = bad
    hx = pu.host_inputs(x)
    args = (sh, hx["q"], hx["k_pool"], hx["v_pool"], hx["page_table"])
    if what[0] in "kv":
        ro, rlse = orc.attn_fwd(*args, osel, ocnt)
        _same_where_finite("O", pu.f32(o), ro, w.dtype)
        _same_where_finite("LSE", pu.f32(lse), rlse, w.dtype)
    glse = lse.cpu().numpy()
    delta = orc.delta(sh, hx["d_o"], pu.f32(o))
    rdq = orc.attn_bwd_dq(*args, glse, delta, hx["d_o"], osel, ocnt)
    rdk, rdv = np.zeros(x["dk_pool"].shape, np.float32), np.zeros(x["dv_pool"].shape, np.float32)
    orc.attn_bwd_dkv(*args, glse, delta, hx["d_o"], rdk, rdv, osel, ocnt)
    dq = attn_bwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], sel, cnt)
    _same_where_finite("dQ", pu.f32(dq), rdq, w.dtype)
    gd = w.dtype if w.grad_dtype == "f32" else "bf16"
    _same_where_finite("dK", pu.f32(x["dk_pool"]), rdk, gd)
    _same_where_finite("dV", pu.f32(x["dv_pool"]), rdv, gd)


@pytest.mark.parametrize("w", [UNSEEN[1], UNSEEN[4], UNSEEN[7]], ids=lambda w: w.name)
def test_what_everyone_sees_reaches_everyone(w):
    # a NaN in a key that every row sees: nothing of the results is finite but the gradients of pages that nobody lists
    x = make_inputs(w, "cuda")
    sel = cnt = None
    if w.top_k is not None:
        sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
    if w.name.startswith("qp_"):
        osel, ocnt = rand_qp_lists(w, w.n_past, w.seed)
        sel, cnt = torch.as_tensor(osel, device="cuda"), torch.as_tensor(ocnt, device="cuda")
    attn_fwd, attn_bwd = (api.paged_attn_fwd_qp, api.paged_attn_bwd_qp) if w.name.startswith("qp_") else (api.paged_attn_fwd, api.paged_attn_bwd)
    for g in range(w.Hkv):
        first = int(sel.reshape(w.Hkv, -1)[g, 0])
        x["k_pool"][x["page_table"][first].long(), g, 0, 0] = math.nan
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, torch_dtype(w.grad_dtype))
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = attn_fwd(*args, sel, cnt)
    dq = attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], sel, cnt)
    assert o.isnan().all() and lse.isnan().all() and dq.isnan().all()
    listed = torch.zeros((w.n_phys, w.Hkv), dtype=torch.bool, device="cuda")
    for g in range(w.Hkv):
        pages = sel.reshape(w.Hkv, -1)[g]
        listed[x["page_table"][pages[pages >= 0].long()].long(), g] = True
    for pool in ("dk_pool", "dv_pool"):
        assert x[pool][listed].isnan().all() and (x[pool][~listed] == 0).all()


@pytest.mark.parametrize("n_past", [1, 40])
def test_rows_whose_scores_are_all_far_below_zero(n_past):
    # products of about -1e33, logits of about -150: a running maximum must not start above them
    w = Workload("low", 4, 2, 64, 16, 32, (n_past + 2) * 16, None, "f32", "f32", 1e-31, seed=120)
    x = make_inputs(w, "cuda")
    x["q"].copy_((1 + x["q"].abs()) * 1e16)
    x["k_pool"].copy_(-(1 + x["k_pool"].abs()) * 1e15)
    hx = pu.host_inputs(x)
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    o, lse = api.paged_attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    ro, rlse = orc.attn_fwd(pu.shape_of(w), hx["q"], hx["k_pool"], hx["v_pool"], hx["page_table"])
    pu.check("O", pu.f32(o), ro, "f32")
    pu.check("LSE", pu.f32(lse), rlse, "f32")
