"""The calls whose speed is watched: whole passes of the paged sparse attention layer over one query chunk.

A pass is what a training or inference loop does per layer and chunk through `paper_2602_02108_amd.api`: (append the chunk's
keys and values,) pick the pages, attention forward, and in training attention backward, with the buffers and
workspaces that such a loop keeps.  A case is a dict of

  select     stream   pooled scores from the past keys themselves, one page list per KV head
             cached   the same from the page means that the paged manager keeps
             votes    softmax votes over the cached means, one page list per query page
             window   the most recent top_k past pages (local-attention layers)
             dense    every page
  append     the chunk's K / V are written to its pages first (with their means, for cached and votes)
  backward   forward and backward, or the forward alone
  offload    K / V and gradient pools in pinned host memory, the listed pages staged
  dtype, grad_dtype, q_heads, kv_heads, head_dim, page, chunk, tokens (history with the chunk), top_k (pages)
"""
import math

import torch

from paper_2602_02108_amd import api
from paper_2602_02108_amd.workloads import Workload, make_inputs, torch_dtype


def _case(name, select, dtype, heads, head_dim, page, chunk, tokens, top_k, grad_dtype="f32", append=False, backward=True,
          offload=False):
    return dict(name=name, select=select, dtype=dtype, grad_dtype=grad_dtype, q_heads=heads[0], kv_heads=heads[1],
                head_dim=head_dim, page=page, chunk=chunk, tokens=tokens, top_k=top_k, append=append, backward=backward,
                offload=offload)


def listed():
    return [
        # the smallest step there is: fp32, small pages, a short history (unit tests, toy models): launches and host work
        _case("fp32_tiny_step", "stream", "f32", (2, 1), 64, 16, 128, 1024, 8),
        # fp32 run of a full-width layer (gradient checks, reference runs)
        _case("fp32_step", "stream", "f32", (28, 4), 128, 128, 512, 16384, 16),
        # a local-attention layer with 64-token pages, ragged page counts, bf16 gradients
        _case("page64_window_step", "window", "bf16", (8, 2), 128, 64, 1088, 19200, 24, grad_dtype="bf16"),
        # inference over small pages and small heads: append, pick, attend
        _case("page16_infer", "cached", "bf16", (14, 2), 64, 16, 512, 32768, 64, append=True, backward=False),
        # inference with a chunk of one page against a long history: few rows, latency counts
        _case("one_page_infer", "cached", "bf16", (28, 4), 128, 128, 128, 131072, 64, append=True, backward=False),
        # a small training step on the matrix kernels
        _case("small_step", "stream", "bf16", (14, 2), 128, 128, 256, 2048, 4),
        # dense attention over a short ragged history, three query heads to a KV head, bf16 gradients
        _case("dense_ragged_step", "dense", "bf16", (6, 2), 128, 128, 1152, 11904, 0, grad_dtype="bf16", append=True),
        # everything in host memory but what the chunk attends
        _case("offload_128k_step", "cached", "bf16", (28, 4), 128, 128, 2048, 131072, 64, offload=True),
        # dense attention over a 64K history
        _case("dense_64k_step", "dense", "bf16", (28, 4), 128, 128, 4096, 65536, 0),
        # 1M history, one list per query page
        _case("votes_1m_step", "votes", "bf16", (28, 4), 128, 128, 4096, 1048576, 128, append=True),
        # 1M history, one list per KV head: the headline workload
        _case("sparse_1m_step", "stream", "bf16", (28, 4), 128, 128, 4096, 1048576, 128),
        # 4M history, the longest chunk and list, bf16 gradients
        _case("sparse_4m_step", "stream", "bf16", (28, 4), 128, 128, 8192, 4194304, 256, grad_dtype="bf16"),
    ]


# Largest work of a drawn case: that of the largest listed case of its kind.
_MAX_FLOPS = {"matrix": 1.5e13, "plain": 6e10}


def draw(rng):
    """One more case of the same ranges."""
    def spread(lo, hi):  # over the logarithm, ends included
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        kind = rng.choice(["step", "step", "step", "infer", "small_pages", "fp32", "offload"])
        backward, append, offload, dtype = True, rng.random() < 0.5, False, "bf16"
        select = rng.choice(["stream", "cached", "votes", "window", "dense"])
        if kind in ("step", "infer"):
            heads, head_dim, page = rng.choice([(28, 4), (28, 4), (14, 2), (6, 2), (32, 8), (4, 4)]), 128, 128
            m, n_past, top_k = spread(1, 64), spread(8, 32704), spread(4, 256)
            if kind == "infer":
                backward, append, m = False, True, spread(1, 16)
            if select == "dense":
                m, n_past = min(m, 32), spread(8, 480)
        elif kind == "offload":
            select, offload, append = rng.choice(["stream", "cached", "votes"]), True, False
            select = "cached" if select == "stream" else select  # (the keys are not on the device)
            heads, head_dim, page = (28, 4), 128, 128
            m, n_past, top_k = spread(1, 32), spread(64, 2016), spread(8, 96)
        else:
            heads, head_dim = rng.choice([(28, 4), (14, 2), (8, 2), (2, 1)]), rng.choice([64, 128])
            page = rng.choice([16, 32, 64]) if kind == "small_pages" else rng.choice([16, 32, 64, 128])
            dtype = "bf16" if kind == "small_pages" else "f32"
            select = rng.choice(["stream", "cached", "window", "dense"])
            backward = rng.random() < 0.7
            m, n_past, top_k = spread(128, 2048) // page, spread(512, 65536) // page, spread(4, 128)
            m = max(1, m)
            if select == "dense":
                n_past = min(n_past, 8192 // page)
        if select in ("window", "dense") and not backward:
            append = True
        top_k = 0 if select == "dense" else min(top_k, n_past)
        c = _case("", select, dtype, heads, head_dim, page, m * page, (m + n_past) * page, top_k,
                  grad_dtype=rng.choice(["f32", "bf16"]), append=append, backward=backward, offload=offload)
        del c["name"]
        plain = dtype == "f32" or page != 128 or head_dim != 128
        if work(c)["flops"] <= _MAX_FLOPS["plain" if plain else "matrix"]:
            return c


def prepare(case, seed):
    """Inputs of the repository's own recipe (N(0, 1) values, shuffled pages, 5 % of the past pages with shifted keys) and the
    buffers and workspaces that a loop over chunks keeps."""
    c = case
    dev = torch.device("cuda:0")
    w = Workload("case", c["q_heads"], c["kv_heads"], c["head_dim"], c["page"], c["chunk"], c["tokens"],
                 None if c["select"] == "dense" else c["top_k"], c["dtype"], c["grad_dtype"], 1.0 / math.sqrt(c["head_dim"]),
                 extra_phys=4, boost_frac=0.05, boost_run=8 if c["tokens"] > 2097152 else 1, seed=seed)
    s = make_inputs(w, dev, zero_grad_pools=c["backward"])
    s.update(case=c, scale=w.sm_scale, gdt=torch_dtype(c["grad_dtype"]), top_k=c["top_k"])
    desc = api.make_desc(s["q"], s["k_pool"], w.N, w.sm_scale, s["gdt"])

    def space(op, k):
        return torch.empty(max(api.workspace_bytes(desc, k, op), 256), dtype=torch.uint8, device=dev)

    def ints(*shape):
        return torch.empty(shape, dtype=torch.int32, device=dev)

    k, votes = c["top_k"], c["select"] == "votes"
    list_k = -1 if c["select"] == "dense" else k
    if c["select"] in ("cached", "votes"):
        s["kbar"] = torch.zeros((w.n, w.Hkv, w.D), dtype=torch.float32, device=dev)
        api.page_means(desc, s["k_pool"], s["page_table"], 0, w.n, s["kbar"])
    if c["select"] != "dense":
        s["sel"] = ints(w.Hkv, w.m, k + w.m) if votes else ints(w.Hkv, k + w.m)
        s["cnt"] = ints(w.Hkv, w.m) if votes else ints(w.Hkv)
    else:
        s["sel"] = s["cnt"] = None
    s["ws_select"] = space(api.OP_VOTE_TOPK if votes else api.OP_SCORE_TOPK, k)
    s["ws_fwd"] = space(api.OP_ATTN_FWD_QP if votes else api.OP_ATTN_FWD, list_k)
    s["o"], s["lse"] = torch.empty_like(s["q"]), torch.empty((w.Hq, w.C), dtype=torch.float32, device=dev)
    if c["backward"]:
        s["ws_bwd"] = space(api.OP_ATTN_BWD_QP if votes else api.OP_ATTN_BWD, list_k)
        s["dq"] = torch.empty_like(s["q"])
    if c["append"]:
        gen = torch.Generator(device=dev)
        gen.manual_seed(seed + 1)
        for name in ("k_chunk", "v_chunk"):
            s[name] = torch.randn((w.C, w.Hkv, w.D), generator=gen, device=dev).to(s["q"].dtype)
    if c["offload"]:
        for name in ("k_pool", "v_pool", "dk_pool", "dv_pool"):
            host = torch.empty(s[name].shape, dtype=s[name].dtype, pin_memory=True)
            host.copy_(s[name])
            s[name] = host
        cap = api.offload_capacity(desc, s["sel"])
        s["plan"] = api.OffloadPlan(desc, cap, dev)
        for name, dt in (("k", s["q"].dtype), ("v", s["q"].dtype), ("dk", s["gdt"]), ("dv", s["gdt"])):
            s["stage_" + name] = torch.zeros((cap,) + tuple(s["k_pool"].shape[1:]), dtype=dt, device=dev)
    return s


def run(state):
    """One pass of the layer over the chunk."""
    s, c = state, state["case"]
    q, table, sel, cnt = s["q"], s["page_table"], s["sel"], s["cnt"]
    desc = api.make_desc(q, s["k_pool"], c["tokens"], s["scale"], s["gdt"])
    kbar = s.get("kbar")
    votes = c["select"] == "votes"
    out = {}
    if c["append"]:
        api.kv_append(desc, s["k_chunk"], s["v_chunk"], table, s["k_pool"], s["v_pool"], kbar)
        out.update(k_pool=s["k_pool"], v_pool=s["v_pool"])
        if kbar is not None:
            out["kbar"] = kbar
    if c["select"] == "stream":
        api.page_score_topk(desc, q, s["k_pool"], table, s["top_k"], sel, cnt, workspace=s["ws_select"])
    elif c["select"] == "cached":
        api.page_score_topk_cached(desc, q, kbar, s["top_k"], sel, cnt, workspace=s["ws_select"])
    elif votes:
        api.page_vote_topk(desc, q, kbar, s["top_k"], sel, cnt, workspace=s["ws_select"])
    elif c["select"] == "window":
        api.local_page_list(desc, s["top_k"], q.device, sel, cnt)
    k_pool, v_pool, dk_pool, dv_pool = s["k_pool"], s["v_pool"], s["dk_pool"], s["dv_pool"]
    if c["offload"]:
        plan = s["plan"]
        api.offload_plan(desc, sel, cnt, plan)
        api.offload_fetch(desc, k_pool, v_pool, table, plan, s["stage_k"], s["stage_v"], s["stage_dk"], s["stage_dv"])
        k_pool, v_pool, dk_pool, dv_pool = s["stage_k"], s["stage_v"], s["stage_dk"], s["stage_dv"]
        host_table, table = table, plan.stage_table
    fwd, bwd = (api.paged_attn_fwd_qp, api.paged_attn_bwd_qp) if votes else (api.paged_attn_fwd, api.paged_attn_bwd)
    fwd(desc, q, k_pool, v_pool, table, sel, cnt, s["o"], s["lse"], s["ws_fwd"])
    out.update(o=s["o"], lse=s["lse"])
    if c["select"] != "dense":
        out.update(sel=sel, cnt=cnt)
    if c["backward"]:
        bwd(desc, q, k_pool, v_pool, table, s["o"], s["lse"], s["d_o"], dk_pool, dv_pool, sel, cnt, s["dq"], s["ws_bwd"])
        out.update(dq=s["dq"], dk_pool=s["dk_pool"], dv_pool=s["dv_pool"])
    if c["offload"]:
        api.offload_writeback(desc, dk_pool, dv_pool, s["dk_pool"], s["dv_pool"], host_table, plan)
    return out


def work(case):
    """Bytes and floating-point operations of one pass: every input read once and every output written once; attention
    products over the visible (query, key) pairs, 4 D per pair forward and 10 D backward."""
    c = case
    es, gs = (2 if c["dtype"] == "bf16" else 4), (2 if c["grad_dtype"] == "bf16" else 4)
    C, D, Hq, Hkv, P = c["chunk"], c["head_dim"], c["q_heads"], c["kv_heads"], c["page"]
    n_past = (c["tokens"] - C) // P
    k = n_past if c["select"] == "dense" else min(c["top_k"], n_past)
    pairs = C * k * P + C * (C + 1) // 2
    held = (k * P + C) * Hkv * D      # elements of K that the chunk attends
    rows = C * Hq * D
    flops = 4.0 * D * pairs * Hq
    size = 2 * held * es + 2 * rows * es + 4 * C * Hq
    if c["backward"]:
        flops += 10.0 * D * pairs * Hq
        size += 3 * rows * es + 2 * held * es + 2 * 2 * held * gs
    if c["select"] == "stream":
        size += n_past * P * D * Hkv * es
        flops += n_past * P * D * Hkv
    elif c["select"] in ("cached", "votes"):
        size += n_past * Hkv * D * 4
        flops += 2.0 * n_past * D * (Hkv if c["select"] == "cached" else C * Hq)
    if c["append"]:
        size += 2 * 2 * C * Hkv * D * es
    return {"bytes": size, "flops": flops}


def tolerance(case):
    """bf16 tensors hold 8 bits; fp32 passes are sums of fp32 products and exponentials.  Page lists from pooled scores are the
    same for every implementation; votes may tie."""
    t = {"rel": 1e-2} if case["dtype"] == "bf16" else {"rel": 1e-2 if case["grad_dtype"] == "bf16" and case["backward"] else 2e-5}
    if case["select"] == "votes":
        t["differ"] = 2e-3
    return t
