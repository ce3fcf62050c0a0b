"""fp32 passes on every route that a call can take: with the workspaces that the library asks for (products in terms, backward by units), without
room for them (the kernels of every shape), and with dQ written over O."""
import math

import pytest
import torch

from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs

import parity_util as pu

pytestmark = pytest.mark.gpu

# heads that do not fill a tile, logits of three times the usual spread (few keys carry a row), keys with a common part
SHAPES = [Workload("d128", 2, 1, 128, 128, 1024, 128 * 40, None, "f32", "f32", 128 ** -0.5, q_scale=3., boost_frac=0.05, seed=501),
          Workload("d64", 6, 2, 64, 32, 800, 32 * 130, None, "f32", "f32", 0.125, q_scale=3., boost_frac=0.05, seed=502)]
ROUTES = [("asked", "asked"), ("asked", "least"), ("none", "asked"), ("none", "least"), ("asked", "over_o")]
PINNED = {"asked": (("fwd_terms",), ()), "none": ((), ("fwd_terms",))}
PINNED_BWD = {"asked": (("bwd_units",), ()), "least": ((), ("bwd_units",)), "over_o": (("bwd_units",), ())}


def exact(w, x):
    """O, LSE, dQ, dK, dV of a dense call in 64 bits, dK / dV as pools."""
    q, d_o = x["q"].double(), x["d_o"].double()
    pages, t = x["page_table"].long()[:w.n], torch.arange(w.N, device="cuda")
    unseen = t[None] > (w.N - w.C + torch.arange(w.C, device="cuda"))[:, None]
    o, dq, lse = torch.zeros_like(q), torch.zeros_like(q), torch.zeros((w.Hq, w.C), dtype=torch.float64, device="cuda")
    dk, dv = (torch.zeros(x["k_pool"].shape, dtype=torch.float64, device="cuda") for _ in range(2))
    for g in range(w.Hkv):
        K, V = (x[n][pages, g].reshape(-1, w.D).double() for n in ("k_pool", "v_pool"))
        dK, dV = torch.zeros_like(K), torch.zeros_like(V)
        for h in range(g * w.G, (g + 1) * w.G):
            S = ((q[:, h] @ K.T) * w.sm_scale).masked_fill(unseen, -math.inf)
            lse[h] = torch.logsumexp(S, 1)
            P = torch.exp(S - lse[h][:, None])
            o[:, h] = P @ V
            dS = P * (d_o[:, h] @ V.T - (d_o[:, h] * o[:, h]).sum(1, keepdim=True))
            dq[:, h] = dS @ K * w.sm_scale
            dK += dS.T @ q[:, h] * w.sm_scale
            dV += P.T @ d_o[:, h]
        dk[pages, g], dv[pages, g] = dK.reshape(-1, w.P, w.D), dV.reshape(-1, w.P, w.D)
    return o, lse, dq, dk, dv


def run(w, x, fwd, bwd):
    """The same from the library, on the route that the workspaces leave."""
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    least = (w.Hq * w.C * 4 + 255) // 256 * 256
    ws = torch.empty(256, dtype=torch.uint8, device="cuda") if fwd == "none" else None
    with pu.kernels_ran(*PINNED[fwd]):
        o, lse = api.paged_attn_fwd(*args, workspace=ws)
    x["dk_pool"].zero_()
    x["dv_pool"].zero_()
    out = o.clone()
    ws = torch.empty(least, dtype=torch.uint8, device="cuda") if bwd == "least" else None
    with pu.kernels_ran(*PINNED_BWD[bwd]):
        dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], d_q=o if bwd == "over_o" else None, workspace=ws)
    return out, lse, dq, x["dk_pool"], x["dv_pool"]


NAMES = ("o", "lse", "dq", "dk", "dv")


def rel(got, want):
    return float((got.double() - want).norm() / want.norm())


# Where forward and backward form S in the same products, what the backward makes of S and LSE carries the errors of the forward's S, and they cancel in dQ.
# Measured, forward with room for splits: O 5.0 to 5.8e-7, dQ 1.0 to 1.7e-6, dK / dV 0.8 to 1.3e-6; without (a row's sums are one chain): O 8.9 to
# 9.6e-7, dQ 1.7 to 2.4e-6, dK / dV 1.0 to 1.4e-6.  With S as fp32 products in both passes O 1.1 to 1.8e-6, dQ 1.6 to 2.6e-6, dK / dV 1.3 to 2.0e-6; in one
# pass only, dQ 3.2 to 4.7e-6, dK / dV up to 2.9e-6.
LIMITS = {"asked": dict(o=9e-7, lse=7e-8, dq=2.1e-6, dk=1.7e-6, dv=1.7e-6), "none": dict(o=1.3e-6, lse=7e-8, dq=2.8e-6, dk=1.7e-6, dv=1.7e-6)}


@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_the_error_does_not_depend_on_the_route(w):
    x = make_inputs(w, "cuda")
    want = exact(w, x)
    for fwd, bwd in ROUTES:
        errs = {n: rel(a, b) for n, a, b in zip(NAMES, run(w, x, fwd, bwd), want)}
        print(w.name, fwd, bwd, {n: f"{e:.2e}" for n, e in errs.items()}, flush=True)
        assert all(errs[n] <= LIMITS[fwd][n] for n in NAMES), (fwd, bwd, errs)


# Keys at the edge of fp32 that carry weight: their first bf16 term must not be rounded to an infinity.  One dim decides: keys of N(0, 1) 1e38, some at
# 3.4e38, queries of about 2^-100 and a scale that makes the logits N(0, 1).  An infinity shows as one, a lost second term as 2^-9; the keys of either sign
# cancel in dQ, whose chains of up to 5120 additions are sqrt(5120) 2^-24 = 4e-6 of their terms off: the line is 2e-5.
@pytest.mark.parametrize("fwd,bwd", ROUTES)
@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_values_at_the_edge_of_fp32_that_carry_weight(w, fwd, bwd):
    w = w.with_(sm_scale=2. ** 100 / 1e38, boost_frac=0., q_scale=1.)
    x = make_inputs(w, "cuda")
    x["q"].mul_(2. ** -100)
    x["d_o"].mul_(2. ** -10)   # (dQ is summed before it is scaled: dS times such a key has to stay finite)
    x["k_pool"][..., 0] = (x["k_pool"][..., 0] * 1e38).clamp_(-3.4e38, 3.4e38)
    x["k_pool"][:, :, 5, 0] = 3.4e38
    x["k_pool"][:, :, 11, 0] = -3.4028e38
    for n, a, b in zip(NAMES, run(w, x, fwd, bwd), exact(w, x)):
        if n != "dk":   # (dS / K: below what fp32 holds)
            assert rel(a, b) <= 2e-5, (n, rel(a, b))


# Values that are not finite, on either route: as they reach those who see them there.
@pytest.mark.parametrize("fwd,bwd", [("none", "least"), ("asked", "asked")])
@pytest.mark.parametrize("what", ["huge", "weight_0", "inf", "nan"])
@pytest.mark.parametrize("w", SHAPES, ids=lambda w: w.name)
def test_values_that_are_not_finite(w, what, fwd, bwd):
    w = w.with_(q_scale=1.)
    x = make_inputs(w, "cuda")
    page, k, q = x["page_table"][w.n_past // 2].long(), x["k_pool"], x["q"]
    hit = torch.zeros((w.C, w.Hq), dtype=torch.bool, device="cuda")   # rows that take up the value
    if what == "huge":
        k[page, :, 3, 0] = 3.4e38
        q[..., 0] = -1
    elif what == "weight_0":
        k[page, :, 3, 0] = -math.inf
        q[..., 0].abs_().add_(0.01)
    elif what == "inf":
        q[100, 1, 5] = math.inf
        hit[100, 1] = True
    else:   # (the rows before it do not see it)
        k[x["page_table"][w.n - 2].long(), 0, 3, 7] = math.nan
        hit[:, :w.G] = (w.N - w.C + torch.arange(w.C, device="cuda") >= (w.n - 2) * w.P + 3)[:, None]
    got, want = run(w, x, fwd, bwd), exact(w, x)
    assert torch.equal(want[0].isnan().any(2), hit)
    assert torch.equal(got[0].isnan().all(2), hit) and torch.equal(got[1].isnan(), hit.T)
    assert rel(got[0][~hit], want[0][~hit]) <= 5e-6 and rel(got[1][~hit.T], want[1][~hit.T]) <= 5e-6
    if what == "huge":
        for n, a, b in zip(NAMES[2:], got[2:], want[2:]):
            assert rel(a, b) <= 5e-6, n
    elif what != "weight_0":
        # dQ of those rows, and dK, dV of every key that one of them sees (of page pg and before it all do, of the pages after it none or some)
        pages = x["page_table"].long()[:w.n]
        seen = pages if what == "nan" else pages[:w.n_past + 100 // w.P]
        clear = torch.ones((w.n_phys, w.Hkv), dtype=torch.bool, device="cuda")
        clear[seen, 0] = False
        ok = ~hit & want[2].isfinite().all(2)   # (the reference multiplies an unseen NaN by 0)
        assert torch.equal(got[2].isnan().all(2), hit) and got[2][~hit].isfinite().all() and (not ok.any() or rel(got[2][ok], want[2][ok]) <= 5e-6)
        assert got[3][seen, 0].isnan().all() and got[4][seen[:w.n_past], 0].isnan().all()
        clear[pages[w.n_past:], 0] = False
        assert not clear.any() or (rel(got[3][clear], want[3][clear]) <= 5e-6 and rel(got[4][clear], want[4][clear]) <= 5e-6)


# Tensors that are small throughout: what the results depend on linearly keeps 24 bits down to the smallest normal value, 2^-126 (as three bf16 terms without
# more: down to 2^-109; at 2^-117 they would be 4e-6 off, at 2^-121 7e-5), also where two of them together make dS small.  The line is that of values of
# the usual size.  Where dO V passes 2^96 the sums overflow on the way and are formed once more from fp32 products: the tolerance of fp32.
@pytest.mark.parametrize("fwd,bwd", [("asked", "asked"), ("none", "least")])
@pytest.mark.parametrize("v_exp,do_exp", [(-117, 0), (0, -117), (-58, -58), (-110, 90), (85, 0), (0, 85), (105, 0)])
@pytest.mark.parametrize("w", [SHAPES[0].with_(C=384, N=128 * 24), SHAPES[1].with_(N=32 * 130)], ids=lambda w: w.name)
def test_tensors_of_any_size_keep_their_bits(w, v_exp, do_exp, fwd, bwd):
    x = make_inputs(w, "cuda")
    x["v_pool"].mul_(2. ** v_exp)
    x["d_o"].mul_(2. ** do_exp)
    errs = {n: rel(a, b) for n, a, b in zip(NAMES, run(w, x, fwd, bwd), exact(w, x))}
    print(w.name, v_exp, do_exp, fwd, bwd, {n: f"{e:.2e}" for n, e in errs.items()}, flush=True)
    if fwd == "asked":
        assert all(errs[n] <= (2e-5 if v_exp == 105 else LIMITS[fwd][n]) for n in NAMES), errs


# dQ is linear in K as well: small keys, keys whose upper dims are small (dQ of each half by itself), and keys of the usual size among which every 128 have one small value.
@pytest.mark.parametrize("fwd,bwd", [("asked", "asked"), ("none", "least")])
@pytest.mark.parametrize("k_exp,do_exp,what", [(-108, 0, "all"), (-117, 30, "all"), (-125, 40, "all"), (-117, 30, "half"), (-125, 30, "few")])
@pytest.mark.parametrize("w", [SHAPES[0].with_(C=384, N=128 * 24), SHAPES[1].with_(N=32 * 130)], ids=lambda w: w.name)
def test_small_keys_keep_their_bits(w, k_exp, do_exp, what, fwd, bwd):
    x = make_inputs(w, "cuda")
    x["d_o"].mul_(2. ** do_exp)
    half = w.D // 2 if what == "half" else w.D
    if what == "few":
        x["k_pool"][:, :, 3, 5] *= 2. ** k_exp
    else:
        x["k_pool"][..., w.D - half:] *= 2. ** k_exp
    got, want = run(w, x, fwd, bwd), exact(w, x)
    errs = {n: rel(a, b) for n, a, b in zip(NAMES, got, want)}
    for n, d in (("dq lower", slice(0, half)), ("dq upper", slice(w.D - half, w.D))):
        errs[n] = rel(got[2][..., d], want[2][..., d])
    print(w.name, k_exp, what, fwd, bwd, {n: f"{e:.2e}" for n, e in errs.items()}, flush=True)
    assert all(e <= LIMITS[fwd][n[:2] if n[0] == "d" else n] for n, e in errs.items()), errs


# Lists that the passes walk in several launches: the backward because of the room that its workspace leaves for the partial sums of dQ (`units` units of 128
# keys of all heads a launch), the forward where the terms of the listed keys pass 512 MiB.  A last launch that is not full, units of the chunk's own pages
# in it, values that are not finite in a key of an early launch that all rows see, and in one of a later launch that few see.
def room_for(w, units):
    up = lambda x: (x + 255) // 256 * 256
    stages, tiles = (w.C * w.G + 31) // 32, (w.C * w.G + 127) // 128
    slot = w.Hkv * 2 * 128 * w.D * 4
    most = (256 if w.D == 128 else 512) // w.Hkv
    return up(w.Hq * w.C * 4) + up(w.Hkv * stages * 6 * 32 * w.D * 2) + (most + units) * slot + units * tiles * w.Hkv * 128 * 128 * 4


IN_LAUNCHES = [(Workload("d128", 28, 4, 128, 128, 512, 128 * 40, None, "f32", "f32", 128 ** -0.5, boost_frac=0.05, seed=511), 7, 6),
               (Workload("d64", 14, 2, 64, 64, 704, 64 * 61, None, "f32", "bf16", 0.125, boost_frac=0.05, seed=512), 12, 3)]


@pytest.mark.parametrize("what", ["finite", "seen by all", "seen by few"])
@pytest.mark.parametrize("w,units,launches", IN_LAUNCHES, ids=lambda v: getattr(v, "name", str(v)))
def test_backward_in_several_launches(w, units, launches, what):
    x = make_inputs(w, "cuda")
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, x["dk_pool"].dtype)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    want = exact(w, x)
    hit = torch.zeros((w.C, w.Hq), dtype=torch.bool, device="cuda")   # rows that see the value, in the heads of KV head 0
    if what != "finite":
        page = 1 if what == "seen by all" else w.n - 1
        x["v_pool"][x["page_table"][page].long(), 0, w.P // 2, 3] = math.inf
        hit[:, :w.G] = (w.N - w.C + torch.arange(w.C, device="cuda") >= page * w.P + w.P // 2)[:, None]
    o, lse = api.paged_attn_fwd(*args)
    for pool in ("dk_pool", "dv_pool"):
        x[pool].fill_(0.25)
    ws = torch.empty(room_for(w, units), dtype=torch.uint8, device="cuda")
    api.profile_reset()
    api.profile_enable(1)
    dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], workspace=ws)
    torch.cuda.synchronize()
    seen = api.profile_read()
    api.profile_enable(0)
    assert seen["bwd_units"][1] == launches
    lost = torch.zeros((w.n_phys, w.Hkv), dtype=torch.bool, device="cuda")   # Delta of those rows is not finite: dK of every key that they see
    lost[:, 0] = bool(hit.any())
    assert torch.equal(dq.isfinite().all(2), ~hit) and torch.equal(x["dk_pool"].isfinite().all(3).all(2), ~lost) and x["dv_pool"].isfinite().all()
    bf = w.grad_dtype == "bf16"
    for n, a, b in (("dq", dq[~hit], want[2][~hit]), ("dk", x["dk_pool"][~lost], want[3][~lost] + 0.25), ("dv", x["dv_pool"], want[4] + 0.25)):
        err = rel(a, b)
        print(w.name, what, n, f"{err:.2e}", flush=True)
        assert err <= (3e-3 if bf and n != "dq" else 2e-6), (n, err)   # (2^-9 of a bf16 element; fp32 sums as above)


@pytest.mark.parametrize("w", [Workload("d128", 64, 32, 128, 128, 512, 128 * 100, None, "f32", "f32", 128 ** -0.5, seed=513),
                               Workload("d64", 64, 32, 64, 64, 512, 64 * 400, None, "f32", "f32", 0.125, seed=514)], ids=lambda w: w.name)
def test_forward_in_several_launches(w):
    x = make_inputs(w, "cuda")
    x["k_pool"][x["page_table"][3].long(), :, 7, 0] = -math.inf   # (a weight of 0, seen in the first launch)
    x["q"][..., 0].abs_().add_(0.01)
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    api.profile_reset()
    api.profile_enable(1)
    o, lse = api.paged_attn_fwd(desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    torch.cuda.synchronize()
    seen = api.profile_read()
    api.profile_enable(0)
    assert seen["fwd_terms"][1] >= 2 and seen["kv_terms"][1] == seen["fwd_terms"][1]
    pages, unseen = x["page_table"].long()[:w.n], torch.arange(w.N, device="cuda")[None] > (w.N - w.C + torch.arange(w.C, device="cuda"))[:, None]
    for h in range(0, w.Hq, 9):
        K, V = (x[n][pages, h // w.G].reshape(-1, w.D).double() for n in ("k_pool", "v_pool"))
        S = ((x["q"][:, h].double() @ K.T) * w.sm_scale).masked_fill(unseen, -math.inf)
        assert rel(o[:, h], torch.softmax(S, 1) @ V) <= 2e-6 and rel(lse[h], torch.logsumexp(S, 1)) <= 1e-7, h


# Calls large enough that neither rows nor keys are split: the kernels of every shape write O, dQ and the gradient pools themselves.  They are left to calls
# with the least workspace; with dQ over O, Delta is formed beforehand or by the dQ kernel.
UNSPLIT = [Workload("keys_d128", 8, 4, 128, 16, 32, 16 * 1100, None, "f32", "bf16", 0.088, seed=521),
           Workload("rows_d64", 32, 32, 64, 64, 1152, 64 * 20, None, "f32", "f32", 0.125, seed=522),
           Workload("rows_d128", 64, 32, 128, 32, 320, 32 * 40, None, "f32", "f32", 0.088, seed=523),
           Workload("keys_d64", 6, 3, 64, 32, 64, 32 * 1100, None, "f32", "f32", 0.125, seed=524)]


@pytest.mark.parametrize("what", ["plain", "over_o", "beside_o", "v_nan", "q_inf"])
@pytest.mark.parametrize("w", UNSPLIT, ids=lambda w: w.name)
def test_unsplit_kernels_with_the_least_workspace(w, what):
    x = make_inputs(w, "cuda")
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, x["dk_pool"].dtype)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    want = exact(w, x)
    hit, lost = torch.zeros((w.C, w.Hq), dtype=torch.bool, device="cuda"), torch.zeros((w.n_phys, w.Hkv), dtype=torch.bool, device="cuda")
    if what == "v_nan":     # a token of the chunk's last page: the rows before it do not see it
        x["v_pool"][x["page_table"][w.n - 1].long(), 0, w.P // 2, 3] = math.nan
        hit[w.C - w.P // 2:, :w.G] = True
    elif what == "q_inf":   # a row of the chunk's first page: the keys after it are not seen by it
        x["q"][w.P // 2, 0, 5] = math.inf
        hit[w.P // 2, 0] = True
    if hit.any():
        lost[x["page_table"].long()[:w.n if what == "v_nan" else w.n_past + 1], 0] = True   # (dK of the keys that they see)
    big = torch.empty((w.C + 1, w.Hq, w.D), device="cuda")
    o, out = big[:-1], big[1:] if what == "beside_o" else None   # (dQ one row further on than O)
    with pu.kernels_ran(("attn_fwd_generic",), absent=("fwd_terms",)):
        o, lse = api.paged_attn_fwd(*args, o=o, workspace=torch.empty(256, dtype=torch.uint8, device="cuda"))
    assert torch.equal(o.isfinite().all(2), ~hit) and rel(o[~hit], want[0][~hit]) <= 3e-6
    ws = torch.empty((w.Hq * w.C * 4 + 255) // 256 * 256, dtype=torch.uint8, device="cuda")
    with pu.kernels_ran(("attn_bwd_generic",), absent=("bwd_units",)):
        dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], d_q=o if what == "over_o" else out, workspace=ws)
    assert torch.equal(dq.isfinite().all(2), ~hit)
    tol = 3e-3 if w.grad_dtype == "bf16" else 6e-6
    seen_dv = ~lost if what == "q_inf" else torch.ones_like(lost)
    part = torch.zeros_like(lost)
    part[x["page_table"].long()[w.n_past], 0] = bool(hit.any())   # (a page of which the row sees the first half only)
    for n, a, b, ok in (("dk", x["dk_pool"], want[3], ~lost), ("dv", x["dv_pool"], want[4], seen_dv)):
        ok = ok & ~part
        assert a[ok].isfinite().all() and rel(a[ok], b[ok]) <= tol, (n, rel(a[ok], b[ok]))
    assert rel(dq[~hit], want[2][~hit]) <= 6e-6


# More KV heads than compute units (a range per head, all of them longer), and rows enough that one launch takes two units.
@pytest.mark.parametrize("w", [Workload("heads", 300, 300, 64, 16, 224, 16 * 40, None, "f32", "f32", 0.125, seed=531),
                               Workload("heads_d128", 264, 264, 128, 32, 160, 32 * 20, None, "f32", "bf16", 0.088, seed=532),
                               Workload("rows", 32, 2, 128, 128, 8192, 128 * 68, None, "f32", "f32", 0.088, seed=533)], ids=lambda w: w.name)
def test_backward_by_units_of_many_heads_and_rows(w):
    x = make_inputs(w, "cuda")
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, x["dk_pool"].dtype)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(*args)
    with pu.kernels_ran(("bwd_units",), absent=()):
        dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"])
    for n, a, b in zip(NAMES, (o, lse, dq, x["dk_pool"], x["dv_pool"]), exact(w, x)):
        assert rel(a, b) <= (3e-3 if a.dtype == torch.bfloat16 else 2e-6), (n, rel(a, b))
