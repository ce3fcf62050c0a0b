"""Values that show how probabilities are held."""
import math

import pytest
import torch

from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs

pytestmark = pytest.mark.gpu


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
