"""Which kernels a backward takes and how its work is shared out: the one launch of bf16 pages of 128, lists shorter than the plan assumes, workspaces with little room."""
import pytest
import torch

from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs

import parity_util as pu
from test_gpu_fp32_routes import exact, rel

pytestmark = pytest.mark.gpu


def backward(w, x, kernels, absent=()):
    """dQ, dK, dV of a dense call with the workspaces that the library asks for, and the same in 64 bits."""
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale, x["dk_pool"].dtype)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(*args)
    with pu.kernels_ran(kernels, absent=absent):
        dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"])
    return (dq, x["dk_pool"], x["dv_pool"]), exact(w, x)[2:]


# bf16 pages of 128: one launch up to half of the workgroups' number (first row) and, beyond that, where equal splits serve the call.  There dS is formed from
# the fp32 probabilities: dK is then one rounding to bf16 off (1.66e-3 of it, dS) and not two (2.35e-3, P and dS); the line is their geometric mean.
@pytest.mark.parametrize("heads,m,n_past", [((14, 2), 2, 14), ((32, 8), 2, 9), ((64, 8), 1, 11), ((6, 2), 11, 36), ((14, 2), 5, 41), ((8, 2), 4, 41), ((4, 4), 16, 8), ((16, 8), 5, 6),
                                            ((8, 8), 9, 2), ((8, 1), 3, 53)])
def test_one_launch_of_pages_of_128_keeps_dk(heads, m, n_past):
    w = Workload("pair", *heads, 128, 128, 128 * m, 128 * (m + n_past), None, "bf16", "f32", 128 ** -0.5, seed=610 + m)
    got, want = backward(w, make_inputs(w, "cuda"), ("bwd_pair",), ("bwd_dkv_mfma",))
    errs = [rel(a, b) for a, b in zip(got, want)]
    print(heads, m, n_past, [f"{e:.2e}" for e in errs], flush=True)
    assert errs[0] < 5e-3 and errs[1] < 2e-3 and errs[2] < 5e-3


# One list per KV head, shorter than its row and not equally long: the work is shared out for the longest one, so that parts of units and of row tiles lie past the end of a list (the first
# head's is the chunk's own pages and one more).  With the room that is asked for (one launch), a third of it (dQ and dK / dV one after the other, with fewer parts) and the least (none).
LISTS = [(14, 2, 128, 128, 256, 40, (3, 23), "bf16"), (8, 2, 128, 64, 192, 60, (4, 37), "bf16"), (6, 2, 64, 16, 112, 200, (8, 131), "bf16"), (12, 3, 64, 128, 128, 24, (2, 24, 9), "bf16"),
         (4, 2, 64, 64, 192, 50, (4, 33), "f32"), (4, 1, 128, 16, 48, 150, (20,), "f32"), (6, 2, 128, 128, 128, 30, (2, 17), "f32")]


# (Pages with kernels of their own need room for their slices: what is asked for.)
@pytest.mark.parametrize("room,Hq,Hkv,D,P,C,stride,counts,dtype", [(room, *case) for case in LISTS for room in (("asked",) if case[:1] == (14,) else ("asked", "third", "least"))])
def test_lists_shorter_than_their_rows(room, Hq, Hkv, D, P, C, stride, counts, dtype):
    w = Workload("short", Hq, Hkv, D, P, C, (stride + 12) * P, None, dtype, "f32", D ** -0.5, extra_phys=2, seed=620 + stride)
    x = make_inputs(w, "cuda")
    g = torch.Generator().manual_seed(w.seed)
    sel = torch.zeros((Hkv, stride), dtype=torch.int32)
    for h, n in enumerate(counts):
        past = torch.randperm(w.n_past, generator=g)[:n - w.m].sort().values
        sel[h, :n] = torch.cat([past, torch.arange(w.n_past, w.n)]).int()
    cnt = torch.tensor(counts, dtype=torch.int32)
    desc = api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale)
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(*args, sel.cuda(), cnt.cuda())
    asked, least = api.workspace_bytes(desc, stride - w.m, api.OP_ATTN_BWD), (Hq * C * 4 + 255) // 256 * 256
    ws = torch.empty({"asked": asked, "third": least + (asked - least) // 3 // 256 * 256, "least": least}[room], dtype=torch.uint8, device="cuda")
    dq = api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], sel.cuda(), cnt.cuda(), workspace=ws)
    ref = pu.oracle_fwd_bwd(w, pu.host_inputs(x), sel.numpy(), cnt.numpy())
    for name, got, want in (("O", o, ref["o"]), ("dQ", dq, ref["dq"]), ("dK", x["dk_pool"], ref["dk_pool"]), ("dV", x["dv_pool"], ref["dv_pool"])):
        pu.check(name, pu.f32(got), want, dtype)


# A workspace asked for once, for the longest history: shorter ones are cut as they are in one of their own, so the results are the same bits.
@pytest.mark.parametrize("Hq,Hkv,D,P,C,tokens,longest,dtype", [(28, 4, 64, 32, 512, 2048, 9088, "bf16"), (8, 2, 128, 64, 1088, 1472, 18112, "bf16"), (6, 2, 128, 16, 128, 2048, 8192, "bf16"),
                                                                (28, 4, 64, 32, 512, 128, 9088, "bf16"), (8, 8, 64, 32, 128, 1024, 2048, "f32"), (28, 4, 128, 16, 16, 640, 38400, "bf16")])
def test_a_workspace_of_the_longest_history_has_room_for_the_parts_of_shorter_ones(Hq, Hkv, D, P, C, tokens, longest, dtype):
    w = Workload("room", Hq, Hkv, D, P, C, tokens + C, None, dtype, "f32", D ** -0.5, seed=640)
    x = make_inputs(w, "cuda")
    desc, last = (api.make_desc(x["q"], x["k_pool"], w.N, w.sm_scale) for _ in range(2))
    last.ctx_len, last.num_phys_pages = longest + C, (longest + C) // P
    args = (desc, x["q"], x["k_pool"], x["v_pool"], x["page_table"])
    o, lse = api.paged_attn_fwd(*args)
    out = []
    for d in (desc, last):
        x["dk_pool"].zero_()
        x["dv_pool"].zero_()
        ws = torch.empty(api.workspace_bytes(d, -1, api.OP_ATTN_BWD), dtype=torch.uint8, device="cuda")
        out.append([t.clone() for t in (api.paged_attn_bwd(*args, o, lse, x["d_o"], x["dk_pool"], x["dv_pool"], workspace=ws), x["dk_pool"], x["dv_pool"])])
    assert all(torch.equal(a, b) for a, b in zip(*out))


# Row tiles in more than 16 parts, up to the 31 that the lookup holds: few rows against a long list, one row tile and two.  fp32 sums of up to 12K keys: 2e-6; bf16: one rounding of dQ to 8 bits (dS and P keep theirs).
@pytest.mark.parametrize("heads,D,P,m,n_past,dtype", [((1, 1), 64, 16, 1, 61, "f32"), ((1, 1), 64, 16, 1, 181, "f32"), ((4, 4), 128, 128, 1, 12, "f32"), ((1, 1), 64, 32, 1, 370, "bf16"),
                                                       ((1, 1), 64, 32, 5, 361, "bf16")])
def test_row_tiles_in_many_parts(heads, D, P, m, n_past, dtype):
    w = Workload("rows", *heads, D, P, m * P, (m + n_past) * P, None, dtype, "f32", D ** -0.5, seed=650 + n_past)
    got, want = backward(w, make_inputs(w, "cuda"), ("attn_bwd_generic",), ("bwd_units",))
    errs = [rel(a, b) for a, b in zip(got, want)]
    print(heads, D, P, m, n_past, [f"{e:.2e}" for e in errs], flush=True)
    assert errs[0] < (2e-6 if dtype == "f32" else 2.5e-3) and max(errs[1:]) < (2e-6 if dtype == "f32" else 1e-3)
