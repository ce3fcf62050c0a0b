"""GPU parity, element by element against the CPU oracle, at sizes the oracle
finishes in seconds (several tiles, ragged tails, edge cases)."""
import numpy as np
import pytest
import torch

import oracle as orc
from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import WORKLOADS, Workload, make_inputs, to_numpy

import parity_util as pu
from test_gpu_parity_full import _sample_rows as sample_rows
from test_gpu_qp_attention import rand_qp_lists

pytestmark = pytest.mark.gpu


def _show(name, rep):
    print(name, {k: (f"{v[0]:.2e}", f"{v[1]:.2e}") for k, v in rep.items()}, flush=True)


@pytest.mark.parametrize("name", ["tiny_dense", "tiny_sparse"])
def test_tiny_fp32(name):
    rep = pu.full_parity(WORKLOADS[name])
    _show(name, rep)


def test_tiny_fp32_accumulates_into_nonzero_pool():
    rep = pu.full_parity(WORKLOADS["tiny_sparse"], init_grad=1.0)
    _show("tiny_sparse+init", rep)


GENERIC_CASES = [
    # fp32, D=128, three KV heads, top-k larger than what is available on purpose
    Workload("f32_d128", 6, 3, 128, 32, 96, 32 * 21, 50, "f32", "f32", 0.09, extra_phys=2, seed=11),
    # bf16 through the shape-generic kernels (P = 64 has no MFMA kernel), bf16 gradient pool
    Workload("bf16_p64", 8, 2, 128, 64, 192, 64 * 19, 5, "bf16", "bf16", 0.088, extra_phys=3, boost_frac=0.2,
             seed=12),
    # no history at all: the chunk is the whole context
    Workload("f32_nohist", 4, 2, 64, 16, 64, 64, 4, "f32", "f32", 0.125, seed=13),
    # top_k = 0: only the local pages
    Workload("f32_k0", 4, 2, 64, 16, 64, 320, 0, "f32", "f32", 0.125, seed=14),
]


@pytest.mark.parametrize("w", GENERIC_CASES, ids=lambda w: w.name)
def test_generic_kernels(w):
    rep = pu.full_parity(w)
    _show(w.name, rep)


# Edges of the shape-generic kernels: tiles of 128 rows (token * G + head) and of 32 / 64 streamed tokens, list
# tokens that fill neither, split and unsplit rows and keys, the diagonal across 16-token pages.
GENERIC_EDGES = [
    Workload("bf16_d64_p16_g7", 14, 2, 64, 16, 48, 16 * 37, 5, "bf16", "f32", 0.125, extra_phys=3, boost_frac=0.2, seed=61),
    Workload("bf16_d64_p128_one_page", 3, 1, 64, 128, 128, 128, 2, "bf16", "bf16", 0.125, seed=62),
    Workload("bf16_p32_dense", 5, 1, 128, 32, 160, 32 * 23, None, "bf16", "f32", 0.088, extra_phys=1, seed=63),
    Workload("f32_d64_p128", 4, 4, 64, 128, 256, 128 * 9, 3, "f32", "f32", 0.125, seed=64),
    Workload("f32_p16_keys_unsplit", 8, 4, 128, 16, 32, 16 * 1100, None, "f32", "bf16", 0.088, seed=65),
    Workload("f32_p64_rows_unsplit", 32, 32, 64, 64, 1152, 64 * 20, 1, "f32", "f32", 0.125, seed=66),
    Workload("bf16_d64_rows_unsplit", 32, 32, 64, 32, 1152, 32 * 41, 3, "bf16", "f32", 0.125, seed=67),
]


@pytest.mark.parametrize("w", GENERIC_EDGES, ids=lambda w: w.name)
def test_generic_kernel_edges(w):
    with pu.kernels_ran(("attn_fwd_generic", "attn_bwd_generic"), absent=pu.MFMA_KERNELS + pu.SPLIT_KERNELS):
        rep = pu.full_parity(w, init_grad=0.25)
    _show(w.name, rep)


# fp32 where the products are formed in three bf16 terms per value, and dQ, dK and dV in one kernel: ranges of stages that end inside a unit, cover
# several short ones (the chunk's own pages) or start at one's first stage; a last unit or tile of 32 keys that is not full; a last row tile that
# is not; lists shorter than their stride; heads that do not divide 256; one split and many.
UNITS_CASES = [
    Workload("f32_units_g7", 28, 4, 128, 128, 384, 128 * 16, 9, "f32", "f32", 0.088, extra_phys=2, boost_frac=0.2, seed=71),
    Workload("f32_units_p16_local", 8, 2, 128, 16, 544, 16 * 51, 13, "f32", "bf16", 0.088, extra_phys=1, seed=72),
    Workload("f32_units_short_list", 6, 3, 128, 64, 320, 64 * 24, 40, "f32", "f32", 0.088, seed=73),
    Workload("f32_units_nohist", 5, 5, 128, 32, 992, 992, 3, "f32", "f32", 0.088, seed=74),
    Workload("f32_units_p32_dense", 2, 1, 128, 32, 352, 32 * 150, None, "f32", "bf16", 0.088, seed=75),
    Workload("f32_units_d64_g7", 14, 2, 64, 16, 624, 16 * 90, 22, "f32", "f32", 0.125, extra_phys=1, seed=76),
    Workload("f32_units_d64_dense", 3, 3, 64, 128, 1024, 128 * 19, None, "f32", "bf16", 0.125, seed=77),
    Workload("f32_units_d64_many_rows", 32, 8, 64, 64, 1088, 64 * 23, 2, "f32", "f32", 0.125, seed=78),
]


@pytest.mark.parametrize("w", UNITS_CASES, ids=lambda w: w.name)
def test_fp32_passes_in_terms(w):
    with pu.kernels_ran(("kv_terms", "fwd_terms", "row_terms", "bwd_units"), absent=pu.MFMA_KERNELS + pu.SPLIT_KERNELS):
        rep = pu.full_parity(w, init_grad=0.25)
    _show(w.name, rep)


# Against 64 bits: 2.5 to 5.0e-7 here (2-norm; sums of fp32 products 5 to 8e-7).  Without one of the small products of terms a product of two values is 2.5 to
# 2.8e-6 off (rms) at least, which shows as 1.7e-6 in O (test_fp32_terms_bounds.py).
@pytest.mark.parametrize("w", [UNITS_CASES[2], UNITS_CASES[5]], ids=lambda w: w.name)
def test_fp32_terms_hold_24_bits(w):
    x = make_inputs(w, "cuda")
    hx, sh = pu.host_inputs(x), pu.shape_of(w)
    sel, cnt, _ = pu.gpu_select(w, x)
    res = pu.gpu_fwd_bwd(w, x, sel, cnt)
    ref = orc.attn_fwd_bwd(sh, hx["q"], hx["k_pool"], hx["v_pool"], hx["page_table"], hx["d_o"], sel.cpu().numpy(), cnt.cpu().numpy(), prec="f64")
    for name in ("o", "dq", "dk_pool", "dv_pool"):
        rel = pu.errors(pu.f32(res[name]), ref[name])[1]
        print(w.name, name, f"{rel:.2e}", flush=True)
        assert rel <= 8e-7, (name, rel)


# Values at the edges of fp32 where products are formed in terms: what would round to an infinity as bf16, an infinity that gives its key
# a weight of 0 (its terms times those of a finite value are NaN), one that makes a row NaN, and a NaN.
@pytest.mark.parametrize("P", [16, 128])
@pytest.mark.parametrize("D", [64, 128])
@pytest.mark.parametrize("what", ["huge", "weight_0", "inf", "nan"])
def test_fp32_terms_of_values_at_the_edges(D, P, what):
    C, n_past = 512, 2048 // P
    w = Workload("edges", 8, 2, D, P, C, C + n_past * P, None, "f32", "f32", D ** -0.5, seed=79)
    x = make_inputs(w, "cuda")
    page = x["page_table"][n_past // 2].long()
    k, q = x["k_pool"], x["q"]
    if what == "huge":
        k[page, :, 3, 0] = 3.4e38
        q[..., 0] = -1
    elif what == "weight_0":
        k[page, :, 3, 0] = float("-inf")
        q[..., 0].abs_().add_(0.01)
    elif what == "inf":
        q[100, 3, 5] = float("inf")
    else:
        k[page, 1, 3, 7] = float("nan")
    desc = api.make_desc(q, k, w.N, w.sm_scale)
    with pu.kernels_ran(("fwd_terms",), absent=()):
        o, lse = api.paged_attn_fwd(desc, q, k, x["v_pool"], x["page_table"])
    pages = x["page_table"].long()
    mask = torch.arange(w.N)[None] <= (w.N - C + torch.arange(C))[:, None]
    for h in range(w.Hq):
        K, V = (x[n][pages, h // 4].reshape(-1, D).double().cpu() for n in ("k_pool", "v_pool"))
        S = ((q[:, h].double().cpu() @ K.T) * w.sm_scale).masked_fill(~mask, float("-inf"))
        want_o, want_lse = torch.softmax(S, 1) @ V, torch.logsumexp(S, 1)
        bad = torch.isnan(want_o).any(1)
        assert torch.equal(torch.isnan(o[:, h].cpu()).all(1), bad), (h, int(bad.sum()))
        if what in ("huge", "weight_0"):
            assert not bad.any()
        assert pu.errors(o[~bad.cuda(), h].cpu(), want_o[~bad])[1] <= 5e-6 and pu.errors(lse[h].cpu()[~bad], want_lse[~bad])[1] <= 1e-6


# Keys of minus infinity that every row sees with a weight of 0, where products are formed in terms: O and LSE are those of the other keys, with
# partial sums that a second kernel combines and without, and no row is formed once more by a wave of its own (which would take many
# times as long as the pass; the line is drawn at 3).
@pytest.mark.parametrize("w", [Workload("split", 28, 4, 128, 128, 512, 128 * 20, None, "f32", "f32", 0.088, seed=80),
                               Workload("unsplit", 32, 32, 64, 32, 2048, 32 * 80, None, "f32", "f32", 0.125, seed=81)], ids=lambda w: w.name)
def test_fp32_terms_of_keys_at_minus_infinity(w):
    x = make_inputs(w, "cuda")
    q, k = x["q"], x["k_pool"]
    q[..., 0].abs_().add_(0.01)
    desc = api.make_desc(q, k, w.N, w.sm_scale)

    def run():
        with pu.kernels_ran(("fwd_terms",), absent=()):
            api.paged_attn_fwd(desc, q, k, x["v_pool"], x["page_table"])   # (the first call also loads the kernel)
            torch.cuda.synchronize()
            api.profile_reset()
            o, lse = api.paged_attn_fwd(desc, q, k, x["v_pool"], x["page_table"])
            torch.cuda.synchronize()
            return o, lse, api.profile_read()["attn_fwd_generic"][0]

    _, _, plain = run()
    page = x["page_table"][1].long()
    k[page, :, 3, 0] = float("-inf")
    o, lse, ms = run()
    pages, pos = x["page_table"].long(), torch.arange(w.N, device="cuda")
    for h in range(0, w.Hq, 5):
        K, V = (x[n][pages, h // w.G].reshape(-1, w.D).double() for n in ("k_pool", "v_pool"))
        S = ((q[:, h].double() @ K.T) * w.sm_scale).masked_fill(pos[None] > (w.N - w.C + torch.arange(w.C, device="cuda"))[:, None], float("-inf"))
        assert pu.errors(o[:, h].cpu(), (torch.softmax(S, 1) @ V).cpu())[1] <= 5e-6
        assert pu.errors(lse[h].cpu(), torch.logsumexp(S, 1).cpu())[1] <= 1e-6
    print(w.name, f"{plain:.3f} {ms:.3f} ms", flush=True)
    assert ms <= 3 * plain, (ms, plain)


# bf16 tensors of shapes without kernels of their own: probabilities and dS keep 32 bits.  Against 64 bits with the same O and LSE
# in the backward, dK / dV carry the rounding of LSE (about 8: 2.4e-7 relative to a probability) and of the exponent, O and
# dQ only that of their own storage, 2^-8 of an element at most.  Probabilities rounded to bf16 miss both by a factor of 100.
@pytest.mark.parametrize("D,P,m,n,top_k", [(64, 16, 3, 37, 5), (64, 128, 1, 6, None), (128, 32, 5, 23, None), (128, 64, 17, 60, 24), (64, 32, 36, 60, 12)])
def test_bf16_shapes_without_kernels_of_their_own_keep_fp32_probabilities(D, P, m, n, top_k):
    w = Workload("wide", 8, 2, D, P, m * P, n * P, top_k, "bf16", "f32", D ** -0.5, extra_phys=2, boost_frac=0.1, seed=80 + m)
    x = make_inputs(w, "cuda")
    hx, sh = pu.host_inputs(x), pu.shape_of(w)
    sel = cnt = osel = ocnt = None
    if top_k is not None:
        sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
        osel, ocnt = sel.cpu().numpy(), cnt.cpu().numpy()
    got = pu.gpu_fwd_bwd(w, x, sel, cnt)
    args = (sh, hx["q"], hx["k_pool"], hx["v_pool"], hx["page_table"])
    o, lse = orc.attn_fwd(*args, osel, ocnt, prec="f64")
    assert np.abs(pu.f32(got["lse"]) - lse).max() <= 4e-6
    glse = got["lse"].cpu().numpy().astype(np.float64)
    delta = orc.delta(sh, hx["d_o"], to_numpy(got["o"].float()), prec="f64")
    dq = orc.attn_bwd_dq(*args, glse, delta, hx["d_o"], osel, ocnt, prec="f64")
    dk, dv = np.zeros(x["dk_pool"].shape), np.zeros(x["dv_pool"].shape)
    orc.attn_bwd_dkv(*args, glse, delta, hx["d_o"], dk, dv, osel, ocnt, prec="f64")
    for name, a, b in (("dK", got["dk_pool"], dk), ("dV", got["dv_pool"], dv)):
        assert pu.errors(pu.f32(a), b)[1] <= 4e-6, (name, pu.errors(pu.f32(a), b))
    for name, a, b in (("O", got["o"], o), ("dQ", got["dq"], dq)):
        over = np.abs(pu.f32(a) - b) - 2.0**-8 * np.abs(b)
        assert over.max() <= 4e-6 * np.abs(b).max(), (name, over.max(), np.abs(b).max())


def test_strided_views_are_honoured():
    """Q / O / dO / dQ as slices of a wider buffer and pools with padded rows."""
    w = WORKLOADS["tiny_sparse"]
    x = make_inputs(w, "cuda")
    hx = pu.host_inputs(x)

    def widen(t, pad):
        shape = list(t.shape)
        shape[-2 if t.dim() == 3 else -1] += 0
        big = torch.zeros(t.shape[:-1] + (t.shape[-1] + pad,), dtype=t.dtype, device=t.device)
        big[..., :t.shape[-1]] = t
        return big[..., :t.shape[-1]]

    xs = dict(x)
    for k in ("q", "d_o", "k_pool", "v_pool", "dk_pool", "dv_pool"):
        xs[k] = widen(x[k], 8)
        assert not xs[k].is_contiguous()
    osel, ocnt, _ = pu.oracle_select(w, hx)
    sel, cnt, _ = pu.gpu_select(w, xs)
    torch.cuda.synchronize()
    assert np.array_equal(sel.cpu().numpy(), osel)
    desc = api.make_desc(xs["q"], xs["k_pool"], w.N, w.sm_scale, torch.float32)
    o = widen(torch.empty_like(x["q"]), 8)
    dq = widen(torch.empty_like(x["q"]), 8)
    o, lse = api.paged_attn_fwd(desc, xs["q"], xs["k_pool"], xs["v_pool"], xs["page_table"], sel, cnt, o=o)
    api.paged_attn_bwd(desc, xs["q"], xs["k_pool"], xs["v_pool"], xs["page_table"], o, lse, xs["d_o"],
                       xs["dk_pool"], xs["dv_pool"], sel, cnt, d_q=dq)
    torch.cuda.synchronize()
    ref = pu.oracle_fwd_bwd(w, hx, osel, ocnt)
    pu.check("O", pu.f32(o), ref["o"], "f32")
    pu.check("dQ", pu.f32(dq), ref["dq"], "f32")
    pu.check("dK", pu.f32(xs["dk_pool"]), ref["dk_pool"], "f32")
    pu.check("dV", pu.f32(xs["dv_pool"]), ref["dv_pool"], "f32")


def test_strided_views_are_honoured_by_the_mfma_kernels():
    """The same with bf16 tensors (MFMA kernels: page images of the forward, direct global -> LDS copies of
    pool rows and of Q / dO rows in the backward): Q / O / dO / dQ rows and pool rows padded by 8 elements,
    bf16 gradient pool."""
    w = Workload("bf16_strided", 14, 2, 128, 128, 256, 128 * 11, 3, "bf16", "bf16", 0.0884, extra_phys=2, seed=41)
    x = make_inputs(w, "cuda")
    hx = pu.host_inputs(x)

    def widen(t, pad=8):
        big = torch.zeros(t.shape[:-1] + (t.shape[-1] + pad,), dtype=t.dtype, device=t.device)
        big[..., :t.shape[-1]] = t
        return big[..., :t.shape[-1]]

    xs = dict(x)
    for k in ("q", "d_o", "k_pool", "v_pool", "dk_pool", "dv_pool"):
        xs[k] = widen(x[k])
        assert not xs[k].is_contiguous()
    osel, ocnt, _ = pu.oracle_select(w, hx)
    sel, cnt, _ = pu.gpu_select(w, xs)
    torch.cuda.synchronize()
    assert np.array_equal(sel.cpu().numpy(), osel)
    desc = api.make_desc(xs["q"], xs["k_pool"], w.N, w.sm_scale, torch.bfloat16)
    o = widen(torch.empty_like(x["q"]))
    dq = widen(torch.empty_like(x["q"]))
    o, lse = api.paged_attn_fwd(desc, xs["q"], xs["k_pool"], xs["v_pool"], xs["page_table"], sel, cnt, o=o)
    api.paged_attn_bwd(desc, xs["q"], xs["k_pool"], xs["v_pool"], xs["page_table"], o, lse, xs["d_o"],
                       xs["dk_pool"], xs["dv_pool"], sel, cnt, d_q=dq)
    torch.cuda.synchronize()
    ref = pu.oracle_fwd_bwd(w, hx, osel, ocnt)
    pu.check("O", pu.f32(o), ref["o"], "bf16")
    pu.check("dQ", pu.f32(dq), ref["dq"], "bf16")
    pu.check("dK", pu.f32(xs["dk_pool"]), ref["dk_pool"], "bf16")
    pu.check("dV", pu.f32(xs["dv_pool"]), ref["dv_pool"], "bf16")


def test_mfma_backward_is_deterministic():
    """bf16 path (sliced dK/dV with the fixed-order reduce): two runs give identical bits."""
    w = WORKLOADS["mid_sparse_bf16"]
    outs = []
    for _ in range(2):
        x = make_inputs(w, "cuda")
        sel, cnt, _ = pu.gpu_select(w, x)
        r = pu.gpu_fwd_bwd(w, x, sel, cnt)
        outs.append({k: v.clone() for k, v in r.items()})
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k


def test_backward_is_deterministic():
    """Page ownership instead of atomics: two runs give identical bits."""
    w = WORKLOADS["tiny_sparse"]
    outs = []
    for _ in range(2):
        x = make_inputs(w, "cuda")
        sel, cnt, _ = pu.gpu_select(w, x)
        r = pu.gpu_fwd_bwd(w, x, sel, cnt)
        outs.append({k: v.clone() for k, v in r.items()})
    for k in outs[0]:
        assert torch.equal(outs[0][k], outs[1][k]), k


@pytest.mark.parametrize("name", ["smoke_bf16", "mid_sparse_bf16", "mid_dense_bf16"])
def test_mfma_bf16(name):
    rep = pu.full_parity(WORKLOADS[name])
    _show(name, rep)


def test_mfma_bf16_nonzero_pool_and_single_local_page():
    # chunk of one page, history of three pages, G = 1
    w = Workload("bf16_g1", 2, 2, 128, 128, 128, 512, 2, "bf16", "f32", 0.0884, seed=31)
    rep = pu.full_parity(w, init_grad=0.5)
    _show(w.name, rep)


# Stage counts of the dK/dV kernel around its ring of four stage buffers (a slice of a page visits
# (C / 32) G / 2 / n_split 64-row stages, fewer on the causal diagonal): slices of 0 / 1 stages, of 1 / 2,
# of 5 (the ring wraps), and two stages per workgroup with the pool updated in place (one slice).
RING_CASES = [
    Workload("bf16_ring_1", 4, 4, 128, 128, 256, 128 * 8, 2, "bf16", "f32", 0.0884, seed=51),
    Workload("bf16_ring_1_2", 6, 2, 128, 128, 128, 128 * 5, None, "bf16", "bf16", 0.0884, seed=52),
    Workload("bf16_ring_5", 2, 1, 128, 128, 640, 128 * 9, 2, "bf16", "f32", 0.0884, seed=53),
    Workload("bf16_ring_in_place", 4, 4, 128, 128, 128, 128 * 512, None, "bf16", "f32", 0.0884, seed=54),
]


# Rows split over workgroups (forward, dQ of bf16 pages of 128): one query page against many splits of two wave
# groups, splits of a single tile, an uneven share, and a list shorter than its row (top_k beyond the history).
SPLIT_CASES = [
    Workload("bf16_split_pairs", 14, 2, 128, 128, 128, 128 * 40, 30, "bf16", "f32", 0.0884, boost_frac=0.1, seed=71),
    Workload("bf16_split_tiles", 3, 1, 128, 128, 128, 128 * 4, 2, "bf16", "bf16", 0.0884, seed=72),
    Workload("bf16_split_uneven", 10, 2, 128, 128, 384, 128 * 23, None, "bf16", "f32", 0.0884, seed=73),
    Workload("bf16_split_short_list", 7, 1, 128, 128, 256, 128 * 5, 9, "bf16", "f32", 0.0884, seed=74),
]


@pytest.mark.parametrize("w", SPLIT_CASES, ids=lambda w: w.name)
def test_mfma_bf16_split_rows(w):
    with pu.kernels_ran(("attn_fwd_split",), absent=("attn_fwd_mfma", "bwd_dq_mfma") + pu.GENERIC_KERNELS):
        rep = pu.full_parity(w, init_grad=0.25)
    _show(w.name, rep)


def _backward_with_dq_over_the_next_row_of_o(w, pad=0):
    """Short calls of bf16 pages of 128 reach the kernels for many rows where dQ overlaps O: dQ one row further on than O.
    pad: elements between the rows of Q / O / dO / dQ and of the pools."""
    x = make_inputs(w, "cuda")
    hx = pu.host_inputs(x)
    gen = torch.Generator(device="cuda").manual_seed(w.seed + 77)
    for k in ("dk_pool", "dv_pool"):
        x[k].copy_((torch.randn(x[k].shape, generator=gen, device="cuda") * 0.25).to(x[k].dtype))
    dk0, dv0 = pu.f32(x["dk_pool"]), pu.f32(x["dv_pool"])
    for k in ("q", "d_o", "k_pool", "v_pool", "dk_pool", "dv_pool"):
        x[k] = torch.empty(x[k].shape[:-1] + (w.D + pad,), dtype=x[k].dtype, device="cuda")[..., :w.D].copy_(x[k])
    sel = cnt = osel = ocnt = None
    if w.top_k is not None:
        sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
        osel, ocnt = sel.cpu().numpy(), cnt.cpu().numpy()
    both = torch.empty((w.C + 1, w.Hq, w.D + pad), dtype=torch.bfloat16, device="cuda")
    o, dq = both[:-1, :, :w.D], both[1:, :, :w.D]
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, x["dk_pool"].dtype)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    _, lse = api.paged_attn_fwd(*args, sel, cnt, o=o)
    with pu.kernels_ran(("bwd_prep", "bwd_dq_mfma", "bwd_dkv_mfma")):
        api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], sel, cnt, d_q=dq)
    ref = pu.oracle_fwd_bwd(w, hx, osel, ocnt, dk0, dv0)
    pu.check("dQ", pu.f32(dq), ref["dq"], "bf16")
    pu.check("dK", pu.f32(x["dk_pool"]), ref["dk_pool"], "bf16")
    pu.check("dV", pu.f32(x["dv_pool"]), ref["dv_pool"], "bf16")


@pytest.mark.parametrize("w", RING_CASES, ids=lambda w: w.name)
def test_mfma_bf16_stage_ring_edges(w):
    _backward_with_dq_over_the_next_row_of_o(w)


@pytest.mark.parametrize("pad", [0, 8])
@pytest.mark.parametrize("w", [WORKLOADS["mid_sparse_bf16"], WORKLOADS["mid_dense_bf16"],
                               Workload("bf16_g1_one_page", 2, 2, 128, 128, 128, 512, 2, "bf16", "f32", 0.0884, seed=31),
                               Workload("bf16_g7", 14, 2, 128, 128, 256, 128 * 11, 3, "bf16", "bf16", 0.0884, extra_phys=2, seed=41)], ids=lambda w: w.name)
def test_mfma_bf16_backward_kernels_for_many_rows(w, pad):
    _backward_with_dq_over_the_next_row_of_o(w, pad)


# The forward kernel for many rows at its edges: last row tile of half its blocks or whole, two to seven query heads
# per KV head.  Oracle rows: page and block boundaries and random ones.
FULL_ROWS = [
    Workload("bf16_rows_g7", 28, 4, 128, 128, 128 * 17, 128 * 70, None, "bf16", "f32", 0.0884, extra_phys=1, seed=76),
    Workload("bf16_rows_g3", 48, 16, 128, 128, 128 * 20, 128 * 80, None, "bf16", "f32", 0.0884, seed=77),
    Workload("bf16_rows_g5_ragged", 20, 4, 128, 128, 128 * 25, 128 * 120, None, "bf16", "f32", 0.0884, seed=78),
    Workload("bf16_rows_g7_sparse", 14, 2, 128, 128, 128 * 33, 128 * 200, 39, "bf16", "f32", 0.0884, boost_frac=0.05, seed=79),
]


def _check_forward_rows(w, x, o, lse, osel, ocnt):
    hx, rows = pu.host_inputs(x), sample_rows(w, 300, w.seed)
    ro, rlse = orc.attn_fwd(pu.shape_of(w), hx["q"], hx["k_pool"], hx["v_pool"], hx["page_table"], osel, ocnt, rows=rows)
    pu.check("O", pu.f32(o)[rows[:, 1], rows[:, 0]], ro, "bf16")
    pu.check("LSE", pu.f32(lse)[rows[:, 0], rows[:, 1]], rlse, "bf16")


@pytest.mark.parametrize("w", FULL_ROWS, ids=lambda w: w.name)
def test_mfma_bf16_forward_kernel_for_many_rows(w):
    x = make_inputs(w, "cuda", zero_grad_pools=False)
    sel = cnt = osel = ocnt = None
    if w.top_k is not None:
        sel, cnt, _ = pu.gpu_select(w, x, want_scores=False)
        osel, ocnt = sel.cpu().numpy(), cnt.cpu().numpy()
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    with pu.kernels_ran(("kv_layout", "attn_fwd_mfma")):
        o, lse = api.paged_attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], sel, cnt)
    _check_forward_rows(w, x, o, lse, osel, ocnt)


# One list per query page: images of two and a half lists are cheap enough for the kernel for many rows, or they are not
@pytest.mark.parametrize("m,k,ran", [(64, 64, "attn_fwd_mfma"), (16, 32, "attn_fwd_split")])
def test_forward_with_lists_per_query_page_takes_the_kernel_that_the_rows_ask_for(m, k, ran):
    w = Workload("bf16_qp_rows", 32, 8, 128, 128, 128 * m, 128 * (m + 100), None, "bf16", "f32", 0.0884, seed=82)
    x = make_inputs(w, "cuda", zero_grad_pools=False)
    osel, ocnt = rand_qp_lists(w, k, w.seed, popular=k // 2)
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    other = {"attn_fwd_mfma": "attn_fwd_split", "attn_fwd_split": "attn_fwd_mfma"}[ran]
    with pu.kernels_ran((ran,), absent=(other,) + pu.GENERIC_KERNELS):
        o, lse = api.paged_attn_fwd_qp(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"], torch.as_tensor(osel, device="cuda"),
                                       torch.as_tensor(ocnt, device="cuda"))
    _check_forward_rows(w, x, o, lse, osel, ocnt)


# The one-launch backward has one name and runs once per call; a call that declines it does not carry the name
def test_the_one_launch_backward_is_timed_once():
    w = WORKLOADS["smoke_bf16"]
    x = make_inputs(w, "cuda")
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(*args)
    for d_q, names in ((torch.empty_like(o), ("bwd_pair",)), (o, ("bwd_dq_split", "bwd_dkv_mfma"))):
        with pu.kernels_ran(names, absent=[n for n in pu.SPLIT_KERNELS + pu.MFMA_KERNELS if n not in names]):
            api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], d_q=d_q)
            torch.cuda.synchronize()
            assert all(api.profile_read()[n][1] == 1 for n in names)
