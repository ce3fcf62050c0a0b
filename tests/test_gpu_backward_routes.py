"""Which kernels a backward takes, and what that does to its results: the one launch of bf16 pages of 128."""
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
