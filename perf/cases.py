"""Cases for timing the decode hot path through the package's public entry points.

A case names an operation and the shape of one attention layer's paged cache:

  step      one decode step: the new token of every sequence appended, pages selected, candidates pruned (one call),
            then attention over the kept tokens
  prune     the pruner alone with every token a candidate (no selector in front)
  channels  the channel-sparse token selector, the pruner on its token lists, attention over the kept tokens
  dense     attention over all tokens
  append    a block of K/V rows written to the cache (prefill): bf16 pools, quantised copy, page bounds

Keys and queries follow the shapes used throughout this repository: K, V, q ~ N(0, 1), head_dim 128, pages of 16
tokens, and per query head a share of heavy tokens whose keys are pushed along the query, which spreads the heads from
near-uniform (alpha 0) to peaked attention.
"""
import math
import random

import torch

from paper_2502_02770_amd import binding as B
from paper_2502_02770_amd.cache import DecodeStep, PagedKV

D, PAGE = 128, 16
CHANNELS = 16          # channel-sparse selector: channels of 128 that take part


def _case(name, op, batch, tokens, q_heads=32, kv_heads=8, div=8, p=0.9, bits=4, ragged=False, shuffle=True, heavy=0.005,
          alpha_lo=0.0, alpha_hi=4.0, spans=False, start=0, lens_seed=0):
    c = dict(op=op, batch=batch, tokens=tokens, q_heads=q_heads, kv_heads=kv_heads, div=div, p=p, bits=bits, ragged=ragged,
             shuffle=shuffle, heavy=heavy, alpha_lo=alpha_lo, alpha_hi=alpha_hi, spans=spans, start=start, lens_seed=lens_seed)
    return c if name is None else dict(c, name=name)


def listed():
    return [
        # a single short chat: everything is launch and dependency latency
        _case("step_1x4k", "step", 1, 4096, div=4, p=0.95, shuffle=False, heavy=0.01, alpha_lo=0.5, alpha_hi=3.0),
        # a few requests of odd lengths on a wide model (8 query heads per KV head)
        _case("step_odd_g8", "step", 5, 9001, q_heads=64, div=8, p=0.95, ragged=True, heavy=0.01, lens_seed=3),
        # one long document, answers clustered in a few spans
        _case("step_1x128k", "step", 1, 131072, div=16, p=0.9, shuffle=False, alpha_lo=1.0, spans=True),
        # the ordinary serving batch (the benchmark's shape)
        _case("step_8x32k", "step", 8, 32768),
        # the same cache with the 8-bit estimator copy, at a shorter context
        _case("step_4x16k_8bit", "step", 4, 16384, bits=8),
        # a full serving batch
        _case("step_32x32k", "step", 32, 32768),
        # mixed traffic: 64 sequences of log-uniform lengths
        _case("step_ragged64", "step", 64, 65536, p=0.95, ragged=True, heavy=0.02),
        # a multi-head model: every query head has its own KV head
        _case("step_mha_8x32k", "step", 8, 32768, kv_heads=32),
        # the pruner on top of full attention: every token of a long context is a candidate
        _case("prune_4x256k", "prune", 4, 262144, q_heads=64, p=0.95, shuffle=False, alpha_hi=6.0),
        # the pruner behind a token-level selector
        _case("channels_8x32k", "channels", 8, 32768),
        # dense attention of layers that are not pruned
        _case("dense_8x32k", "dense", 8, 32768),
        # prefill of the serving batch
        _case("append_8x32k", "append", 8, 32768),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    op = rng.choice(["step"] * 8 + ["prune", "channels", "dense", "append"])
    q_heads, kv_heads = rng.choice([(32, 8), (32, 8), (32, 8), (64, 8), (32, 32), (16, 8)])
    # rows (tokens x KV heads) and scores (tokens x query heads) of the largest listed case of the operation
    most = {"step": 1 << 23, "prune": 1 << 23, "channels": 1 << 21, "dense": 1 << 21, "append": 1 << 21}[op]
    scores = {"step": 1 << 25, "prune": 1 << 26, "channels": 1 << 23, "dense": 1 << 24, "append": 1 << 24}[op]
    top = min(most // kv_heads, scores // q_heads)
    batch = _log_int(rng, 1, 64)
    tokens = _log_int(rng, 512, max(1024, min(131072, top // batch)))
    return _case(None, op, batch, tokens, q_heads=q_heads, kv_heads=kv_heads, div=rng.choice([4, 8, 8, 16]),
                 p=rng.choice([0.8, 0.9, 0.95, 0.99]), bits=rng.choice([4, 4, 4, 4, 4, 8, 2]) if op == "step" else 4,
                 ragged=rng.random() < 0.5, shuffle=rng.random() < 0.75, heavy=rng.choice([0.002, 0.005, 0.02]),
                 spans=rng.random() < 0.2, start=rng.randrange(0, 4096) if op == "append" else 0, lens_seed=rng.randrange(1 << 30))


def _lens(case):
    """Valid tokens of each sequence: the case's length, or log-uniform from 1/32 of it (at least 64 tokens) up to it."""
    n, b = case["tokens"], case["batch"]
    if not case["ragged"]:
        return [n] * b
    r = random.Random(case["lens_seed"])
    return [_log_int(r, max(64, n // 32), n) for _ in range(b)]


def _budgets(case):
    return [max(PAGE, n // case["div"]) for n in _lens(case)]


def _tokens(case, g, lens, q):
    """K and V of all sequences, concatenated: [total, kv_heads, 128] bf16, with the heavy tokens of every query head."""
    dev = q.device
    Hkv, G = case["kv_heads"], case["q_heads"] // case["kv_heads"]
    total = sum(lens)
    k = torch.randn(total, Hkv, D, dtype=torch.bfloat16, device=dev, generator=g)
    v = None
    if case["op"] != "prune":
        v = torch.randn(total, Hkv, D, dtype=torch.bfloat16, device=dev, generator=g)
    if case["op"] in ("append", "dense"):
        return k, v
    alpha = case["alpha_lo"] + (case["alpha_hi"] - case["alpha_lo"]) * torch.rand(len(lens), Hkv, G, 1, device=dev, generator=g)
    qf = q.float().view(len(lens), Hkv, G, D)
    push = (alpha * math.sqrt(D) * qf / qf.norm(dim=-1, keepdim=True)).to(torch.bfloat16)
    at = 0
    for b, n in enumerate(lens):
        rows = k[at:at + n]
        for j in range(G):
            if case["spans"]:                   # 8 spans of 64 tokens (shorter in short sequences)
                length = min(64, max(1, n // 16))
                first = torch.randint(0, n - length + 1, (8, Hkv), device=dev, generator=g)
                pos = torch.arange(n, device=dev).view(n, 1, 1)
                mask = ((pos >= first) & (pos < first + length)).any(dim=1)
            else:
                mask = torch.rand(n, Hkv, device=dev, generator=g) < case["heavy"]
            rows.add_(mask.unsqueeze(-1).to(torch.bfloat16) * push[b, :, j])
        at += n
    return k, v


def _i32(values, dev):
    return torch.tensor(values, dtype=torch.int32, device=dev)


def prepare(case, seed):
    dev = torch.device("cuda", torch.cuda.current_device())
    g = torch.Generator(device=dev)
    g.manual_seed(int(seed))
    lens, b = _lens(case), case["batch"]
    Hq, Hkv, op = case["q_heads"], case["kv_heads"], case["op"]
    start = case["start"]
    q = torch.randn(b, Hq, D, dtype=torch.bfloat16, device=dev, generator=g)
    k, v = _tokens(case, g, lens, q)
    offsets = [0]
    for n in lens:
        offsets.append(offsets[-1] + n)

    pages = [(start + n + PAGE - 1) // PAGE for n in lens]
    used = sum(pages)
    perm = torch.randperm(used, device=dev, generator=g) if case["shuffle"] else torch.arange(used, device=dev)
    table = torch.full((b, max(pages)), -1, dtype=torch.int32, device=dev)
    at = 0
    for i, m in enumerate(pages):
        table[i, :m] = perm[at:at + m].to(torch.int32)
        at += m
    cache = PagedKV(Hq, Hkv, table, _i32([start + n for n in lens], dev), used, dev, need_v=v is not None, quant_bits=case["bits"])
    s = dict(op=op, cache=cache, q=q, p=case["p"])

    if op == "append":
        if start:                               # tokens already in the cache, so that the first page is shared
            old = torch.randn(b * start, Hkv, D, dtype=torch.bfloat16, device=dev, generator=g)
            cache.append(old, old, _i32([0] * b, dev), _i32([start] * b, dev), _i32([i * start for i in range(b)], dev), start)
        s.update(k=k, v=v, start=_i32([start] * b, dev), n_new=_i32(lens, dev), offs=_i32(offsets[:-1], dev), max_new=max(lens))
        return s
    # the cache as the previous step left it: everything but the last token, which the step brings
    last = 1 if op == "step" else 0
    cache.append(k, v, _i32([0] * b, dev), _i32([n - last for n in lens], dev), _i32(offsets[:-1], dev), max(lens))
    if op == "step":
        ends = torch.tensor([o - 1 for o in offsets[1:]], device=dev)
        s.update(k_new=k[ends].contiguous(), v_new=v[ends].contiguous(), new_pos=_i32([n - 1 for n in lens], dev))
    if op == "dense":
        s["step"] = DecodeStep(cache, max_sel=1)
        return s
    budgets = _budgets(case)
    s["budget"] = _i32(budgets, dev)
    if op == "prune":
        s["step"] = DecodeStep(cache)
        return s
    most = (max(budgets) + PAGE - 1) // PAGE
    if op == "step":
        s["step"] = DecodeStep(cache, max_sel=most)
        return s
    # channels: token lists of at most 8192 entries
    cand = min(8192, most * PAGE)
    st = DecodeStep(cache, max_sel=cand // PAGE)
    weight = k.float().abs().mean(dim=0) * q.float().abs().mean(dim=0).view(Hkv, Hq // Hkv, D).mean(dim=1)
    chosen = torch.zeros(Hkv, D, dtype=torch.int64, device=dev)
    chosen.scatter_(1, weight.topk(CHANNELS, dim=1).indices, 1)
    words = (chosen.view(Hkv, 4, 32) << torch.arange(32, device=dev)).sum(dim=2)
    s.update(step=st, max_cand=cand, mask=torch.where(words >= 1 << 31, words - (1 << 32), words).to(torch.int32).contiguous(),
             cand=torch.zeros(b, Hq, cand, dtype=torch.int32, device=dev), count=torch.zeros(b, Hq, dtype=torch.int32, device=dev),
             ws_sel=torch.empty(B.twilight_workspace_bytes(B.TW_WS_DS_SELECT, cache.kv, cand), dtype=torch.uint8, device=dev),
             ws_prune=torch.empty(B.twilight_workspace_bytes(B.TW_WS_PRUNE_TOKENS, cache.kv, cand), dtype=torch.uint8, device=dev))
    return s


def _cache_state(c):
    return [c.kq_pool, c.kq_meta, c.page_minmax] + [t for t in (c.k_pool, c.v_pool) if t is not None]


def run(s):
    c, op = s["cache"], s["op"]
    if op == "append":
        c.append(s["k"], s["v"], s["start"], s["n_new"], s["offs"], s["max_new"])
        return _cache_state(c)
    st, q = s["step"], s["q"]
    if op == "dense":
        return [st.dense(q, lse=st.lse), st.lse]
    if op == "prune":
        st.prune(q, s["p"])
        return [st.kept_count, st.union_count, st.union_idx, st.status]
    if op == "step":
        st.select_prune(s["k_new"], s["v_new"], s["new_pos"], q, s["budget"], s["p"])
        st.attend(q)
        return [st.out, st.lse, st.sel_pages, st.sel_count, st.kept_count, st.union_count, st.union_idx, st.status] + _cache_state(c)
    B.twilight_ds_select_tokens(c.kv, q, s["mask"], s["budget"], s["cand"], s["count"], s["max_cand"], s["ws_sel"])
    B.twilight_topp_prune_tokens(c.kv, q, s["cand"], s["count"], s["max_cand"], s["p"], st.kept_count, None, 0, st.union_count,
                                 st.union_idx, st.union_stride, st.status, s["ws_prune"])
    st.attend(q)
    return [st.out, st.lse, s["cand"], s["count"], st.kept_count, st.union_count, st.union_idx, st.status]


def work(case):
    """Bytes and operations of one pass.  Which pages and tokens are read depends on the data: candidate pages of a KV
    head are counted as if its query heads chose them independently, kept tokens as 6 % of a head's candidates."""
    Hq, Hkv, op = case["q_heads"], case["kv_heads"], case["op"]
    G, lens = Hq // Hkv, _lens(case)
    row = 4 * D                                                     # a K row and a V row, bf16
    code = D * case["bits"] / 8 + 16                                # a token's codes and its scales
    total = sum(lens)
    if op == "append":
        return {"bytes": total * Hkv * (2 * row + code + 4 * D / PAGE), "flops": total * Hkv * D * 6}
    if op == "dense":
        return {"bytes": total * Hkv * row, "flops": total * Hq * 4 * D}
    if op == "prune":
        # half of the tokens end up in a group's list
        return {"bytes": total * Hkv * (code + 2), "flops": total * Hq * 2 * D}
    nbytes, flops = 0.0, 0.0
    for n, budget in zip(lens, _budgets(case)):
        share = min(1.0, budget / n)
        kept = min(n, 0.06 * budget * G)
        nbytes += Hkv * (kept * (row + 8) + 4 * D * G)
        flops += Hkv * kept * G * 4 * D
        if op == "step":
            nbytes += Hkv * (n / PAGE * 4 * D + n * (1.0 - (1.0 - share) ** G) * code + 4 * n * share * G / PAGE)
            flops += Hq * (n / PAGE * 2 * D + budget * 2 * D)
        else:
            nbytes += Hkv * (n * code + 8 * budget * G)
            flops += Hq * (n * 2 * CHANNELS + budget * 2 * D)
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    # Lists, counts and cache contents are defined bit for bit.  The attention output is rounded to bf16: against the
    # same sums in 64 bits it is off by 1.6e-3 (2-norm) and 3.9e-3 (largest) over all listed cases; four times that.
    if case["op"] in ("append", "prune"):
        return "exact"
    return {"rel": 6.5e-3, "max": 1.6e-2}
