"""GPU parity at the edges of the kernels' dispatch rules and tiles, against the CPU oracle."""
import numpy as np
import pytest
import torch

from oracle import twilight_oracle as O
from workloads import synth
from tests.gpu_util import assert_attention, build_cache, u16

pytestmark = pytest.mark.gpu


def _T():
    import paper_2502_02770_amd as T
    return T


@pytest.mark.parametrize("P", [1, 2, 64, 256, 257, 512, 513, 2048, 2049, 8192, 8193, 32768, 32769])
def test_page_lists_at_the_row_lengths_of_the_selection_kernels(P):
    """Random page bounds, rows one entry short of, at and beyond the length where the next selection kernel takes
    over, budgets of one page, half of the row and all but one page: page lists bit for bit."""
    T = _T()
    rng = np.random.default_rng(P)
    table = torch.arange(P, dtype=torch.int32).view(1, P)
    n = 16 * P - 3 if P > 1 else 16
    cache = T.PagedKV(2, 1, table, torch.tensor([n]), P, need_v=False)
    mm = torch.from_numpy(np.sort(rng.standard_normal((P, 1, 2, 128)).astype(np.float32), axis=2)).to(torch.bfloat16)
    mm[rng.integers(0, P, size=P // 4)] = mm[0].clone()                    # some pages tie
    cache.page_minmax.copy_(mm)
    q = torch.from_numpy(rng.standard_normal((1, 2, 128)).astype(np.float32)).to(torch.bfloat16)
    for budget in sorted({16, 16 * max(1, P // 2), 16 * max(1, P - 1)}):
        st = T.DecodeStep(cache, max_sel=max(1, budget // 16))
        st.select(q.cuda(), torch.tensor([budget], dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        for h in range(2):
            U = O.page_upper_bounds(synth.bits(q[0, h]), u16(mm[:, 0, 0]), u16(mm[:, 0, 1]))
            want = O.select_pages(U, budget, n)
            assert st.sel_pages[0, h, :int(st.sel_count[0, h])].cpu().numpy().tolist() == want.tolist(), (budget, h)


def _random_bounds(T, lens, max_pages, heads=(32, 8), pool=64, seed=0):
    """Cache whose pages carry random key bounds (pool pages shared by the sequences) and a query."""
    g = torch.Generator().manual_seed(seed)
    table = (torch.arange(len(lens) * max_pages, dtype=torch.int32) % pool).view(len(lens), max_pages)
    cache = T.PagedKV(heads[0], heads[1], table, torch.tensor(lens), pool, need_v=False)
    mm = torch.randn(pool, heads[1], 2, 128, generator=g).sort(dim=2).values.to(torch.bfloat16)
    cache.page_minmax.copy_(mm)
    return cache, torch.randn(len(lens), heads[0], 128, generator=g).to(torch.bfloat16).cuda()


def _selection_us(T, pages, max_pages, batch):
    """Median time of the selection kernels (without the bounds) for `batch` x 32 rows of `pages` entries."""
    B = T.binding
    cache, q = _random_bounds(T, [16 * pages] * batch, max_pages)
    st = T.DecodeStep(cache, max_sel=max(1, pages // 8))
    budget = torch.full((batch,), 2 * pages, dtype=torch.int32, device="cuda")
    for _ in range(3):
        st.select(q, budget)
    torch.cuda.synchronize()
    B.twilight_prof_enable(1)
    for _ in range(15):
        st.select(q, budget)
    torch.cuda.synchronize()
    rec = B.twilight_prof_collect()
    B.twilight_prof_enable(0)
    runs = np.array([ms for _, ms in rec]).reshape(15, -1) * 1e3
    return float(np.median(runs[:, 1:].sum(axis=1)))


def test_short_rows_under_a_long_bound_cost_no_more_than_full_ones():
    """512 rows of 500 entries under a bound of 9000 (most waves of the selection hold no entry at all): the slots
    beyond the row's end must not be bucketed."""
    T = _T()
    short, full = _selection_us(T, 500, 9000, 16), _selection_us(T, 9000, 9000, 16)
    assert short < full, (short, full)


def test_selection_time_follows_the_length_of_the_row():
    """512 rows of a quarter of the bound's length: the selection handles their entries, not the bound's."""
    T = _T()
    short, full = _selection_us(T, 8000, 32768, 16), _selection_us(T, 32768, 32768, 16)
    assert short < 0.55 * full, (short, full)


@pytest.mark.parametrize("max_pages", [2500, 9000, 16384, 16385, 32768])
def test_page_lists_of_short_rows_under_a_long_bound(max_pages):
    """Rows shorter than the bound that chooses the selection kernel, at the lengths where its body or the groups of slots
    that it skips change, down to one with a wave's worth of entries: page lists bit for bit."""
    T = _T()
    pages = [max_pages, 1100, 700, 65, 17, 2] + [P + i for P in (4096, 8192, 12288, 28672) for i in (0, 1) if P + i < max_pages]
    cache, q = _random_bounds(T, [16 * P for P in pages], max_pages, heads=(2, 1), pool=4096, seed=max_pages)
    for cut in (2, 7):
        budget = [16 * max(1, P // cut) for P in pages]
        st = T.DecodeStep(cache, max_sel=max_pages // cut)
        st.select(q, torch.tensor(budget, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        mm = cache.page_minmax.cpu()
        for b, P in enumerate(pages):
            rows = mm[cache.page_table[b, :P].cpu().long(), 0]
            for h in range(2):
                U = O.page_upper_bounds(synth.bits(q[b, h].cpu()), u16(rows[:, 0]), u16(rows[:, 1]))
                want = O.select_pages(U, budget[b], 16 * P)
                assert st.sel_pages[b, h, :int(st.sel_count[b, h])].cpu().numpy().tolist() == want.tolist(), (b, h, cut)


def _prune_us(T, keys, batch, n, heads, p=0.95):
    """Median time of the pruner's kernels with every token a candidate; keys(gen) -> [batch * n, kv_heads, 128]."""
    B = T.binding
    g = torch.Generator(device="cuda").manual_seed(7)
    pages = (n + 15) // 16
    cache = T.PagedKV(heads[0], heads[1], torch.arange(batch * pages, dtype=torch.int32).view(batch, pages),
                      torch.tensor([n] * batch), batch * pages, need_v=False)
    cache.fill(keys(g).to(torch.bfloat16), None, [i * n for i in range(batch + 1)])
    q = torch.randn(batch, heads[0], 128, device="cuda", generator=g).to(torch.bfloat16)
    st = T.DecodeStep(cache)
    for _ in range(3):
        st.prune(q, p)
    torch.cuda.synchronize()
    B.twilight_prof_enable(1)
    for _ in range(9):
        st.prune(q, p)
    torch.cuda.synchronize()
    rec = B.twilight_prof_collect()
    B.twilight_prof_enable(0)
    return float(np.median(np.array([ms for _, ms in rec]).reshape(9, -1).sum(axis=1)) * 1e3)


def test_long_rows_of_equal_keys_are_searched_quickly():
    """Rows whose listed scores overflow (all keys equal, or drawn from four) are searched again from the scores by one
    workgroup per row: that must not take several times what the rest of the pruner takes.  (Every score of such a row
    falls into one bucket, so one LDS add per score makes it a serial chain.)"""
    T = _T()
    n, Hkv = 65536, 2
    plain = _prune_us(T, lambda g: torch.randn(n, Hkv, 128, device="cuda", generator=g), 1, n, (8, Hkv))
    equal = _prune_us(T, lambda g: torch.randn(1, Hkv, 128, device="cuda", generator=g).expand(n, Hkv, 128), 1, n, (8, Hkv))
    few = _prune_us(T, lambda g: torch.randn(4, Hkv, 128, device="cuda", generator=g)[torch.randint(0, 4, (n,), device="cuda", generator=g)], 1, n, (8, Hkv))
    assert equal < 3 * plain and few < 3 * plain, (plain, equal, few)


@pytest.mark.parametrize("p", [0.99999, 0.999999])
def test_long_peaked_rows_with_p_near_one_list_few_scores(p):
    """Logits of deviation 4 and p near 1: what is left out is next to none of the mass - of the size of what the exact masses
    (multiples of 2^-40) drop of every score - but most of the scores.  The scores that the histogram leaves undecided
    must still fit the list and hold the threshold (a row searched again takes several times the whole of top-p)."""
    T = _T()
    n, Hkv = 65536, 8
    keys = lambda g: 4 * torch.randn(n, Hkv, 128, device="cuda", generator=g)
    plain, near = _prune_us(T, keys, 1, n, (64, Hkv), 0.95), _prune_us(T, keys, 1, n, (64, Hkv), p)
    assert near < 1.4 * plain, (plain, near)


def test_query_rows_at_an_odd_element():
    """The scoring and pruning entry points take a query that begins at any bf16 element."""
    T = _T()
    w = synth.make_workload("oddq", [700, 9000], num_q_heads=8, num_kv_heads=2, budget=512, p=0.9, heavy_frac=0.01,
                            alpha_range=(0.0, 3.0), need_v=False, seed=93)
    cache = build_cache(w)
    q = w.q.cuda()
    odd = torch.zeros(q.numel() + 1, dtype=torch.bfloat16, device="cuda")[1:].view(q.shape)
    odd.copy_(q)
    assert odd.data_ptr() % 4 == 2
    full, listed = T.DecodeStep(cache), T.DecodeStep(cache, max_sel=32)
    listed.select(q, w.budget.cuda())
    for st in (full, listed):
        got = []
        for x in (q, odd):
            st.union_idx.fill_(-1)
            st.prune(x, w.p)
            torch.cuda.synchronize()
            got.append([t.clone() for t in (st.kept_count, st.union_count, st.union_idx)])
        assert all(torch.equal(a, b) for a, b in zip(*got))


@pytest.mark.parametrize("batch", [3, 20], ids=["few_lists", "many_lists"])
@pytest.mark.parametrize("G", [1, 2, 4, 8])
def test_attention_over_lists_at_the_edges_of_a_step(G, batch):
    """Lists of every remainder of a wave's 16 and a workgroup's 64 rows, empty ones, one that is cut into many chunks,
    entries that do not count in between; the pool's first page holds NaN and belongs to no sequence.  Few lists: the
    item map in registers, many: through LDS.  Definition 3.1 in float64, the bars of the other attention tests."""
    T = _T()
    H, n = 4, 5000
    rng = np.random.default_rng(100 * G + batch)
    P = (n + 15) // 16
    table = 1 + torch.arange(batch * P, dtype=torch.int32).view(batch, P)
    cache = T.PagedKV(G * H, H, table, torch.full((batch,), n), 1 + batch * P)
    k = torch.from_numpy(rng.standard_normal((batch * n, H, 128)).astype(np.float32)).to(torch.bfloat16)
    v = torch.from_numpy(rng.standard_normal((batch * n, H, 128)).astype(np.float32)).to(torch.bfloat16)
    cache.fill(k.cuda(), v.cuda(), [b * n for b in range(batch + 1)])
    cache.k_pool[0] = float("nan")
    cache.v_pool[0] = float("nan")
    q = torch.from_numpy(rng.standard_normal((batch, G * H, 128)).astype(np.float32)).to(torch.bfloat16)
    lens = ([0, 1, 2, 3, 4, 5, 15, 16, 17, 31, 48, 63, 64, 65, 66, 68, 80, 127, 128, 129, 191, 192, 193, 255, 257, 600] * 4)[:batch * H]
    lens[1], lens[3] = 4900, 1300
    stride = 4928
    idx = np.zeros((batch * H, stride), np.int32)
    for l, c in enumerate(lens):
        idx[l, :c] = np.sort(rng.permutation(n)[:c])
        if c > 4:                                         # entries that do not count: in front, at the end, anywhere
            idx[l, [0, c - 1, int(rng.integers(1, c - 1))]] = [-1, n, 1 << 30]
    st = T.DecodeStep(cache, max_sel=1, union_stride=stride)
    st.union_count.copy_(torch.tensor(lens, dtype=torch.int32))
    st.union_idx.copy_(torch.from_numpy(idx))
    st.attend(q.cuda())
    torch.cuda.synchronize()
    out, lse = st.out.cpu().float().numpy(), st.lse.cpu().numpy()
    for l, c in enumerate(lens):
        b, g = divmod(l, H)
        ids = idx[l, :c][(idx[l, :c] >= 0) & (idx[l, :c] < n)]
        kb, vb = synth.bits(k.view(batch, n, H, 128)[b, :, g]), synth.bits(v.view(batch, n, H, 128)[b, :, g])
        for h in range(g * G, g * G + G):
            if not len(ids):
                assert not out[b, h].any() and np.isneginf(lse[b, h])
                continue
            ref, rl = O.attention(synth.bits(q[b, h]), kb, vb, ids)
            assert_attention(out[b, h].astype(np.float64), ref)
            assert abs(lse[b, h] - rl) <= 1e-3 * max(1.0, abs(rl))


@pytest.mark.parametrize("n,max_sel,seqs,separate", [(16384, 64, 36, False), (32768, 128, 2, False), (65536, 256, 2, False), (65536, 256, 32, False),
                                                     (65536, 512, 32, False), (65536, 512, 36, False), (196608, 512, 1, True)])
def test_kept_tokens_of_the_last_page_reach_the_union(n, max_sel, seqs, separate):
    """Rows of pages that fill the kernel's position bitmap exactly: heavy tokens in all of the last page, which end up
    kept, for every workgroup size; the union is that of the kept lists, the last token included."""
    T = _T()
    w = synth.make_workload("last", [n] + [600] * (seqs - 1), num_q_heads=8, num_kv_heads=2, budget=max_sel * 16, p=0.9999,
                            heavy_frac=0.0, alpha_range=(0.0, 0.0), shuffle_pool=True, need_v=False, seed=96)
    qh = w.q[0].float().view(2, 4, 128)
    push = (qh / qh.norm(dim=-1, keepdim=True)).sum(dim=1) * 11.3
    w.k[n - 16:n] = (w.k[n - 16:n].float() + push).to(torch.bfloat16)
    cache = build_cache(w)
    q, budget = w.q.to(cache.device), w.budget.to(cache.device)
    st = T.DecodeStep(cache, max_sel=max_sel, with_kept_idx=True)
    if separate:
        st.select(q, budget)
        st.prune(q, w.p)
    else:
        st.select_prune(None, None, None, q, budget, w.p)
    torch.cuda.synchronize()
    for g in range(2):
        kept = np.unique(np.concatenate([st.kept_idx[0, h, :int(st.kept_count[0, h])].cpu().numpy() for h in range(4 * g, 4 * g + 4)]))
        assert set(range(n - 16, n)) <= set(kept.tolist())
        assert st.union_idx[g, :int(st.union_count[g])].cpu().numpy().tolist() == kept.tolist()
@pytest.mark.parametrize("bits,heads,lens,max_sel", [
    (4, (8, 2), [131072, 40, 9000], 512), (4, (8, 1), [131065], 511), (4, (16, 16), [66000, 1, 16], 300), (4, (4, 2), [131072] * 2, 257),
    (2, (32, 8), [65536, 20000, 4100], 512), (8, (32, 8), [65536, 20000, 4100], 400), (4, (64, 8), [70001, 300], 512),
    (4, (12, 12), [40000, 2, 70000], 509)])
def test_one_launch_select_prune_of_few_heads_with_long_lists(bits, heads, lens, max_sel):
    """Lists above 4096 candidates on at most half as many heads as CUs: 2 to 8 workgroups per head, with and without a
    multiple of 8 KV groups, lists shorter than the workgroups are many, 8192 pages; twice on the same workspace, against
    the separate calls bit for bit."""
    T = _T()
    w = synth.make_workload("split", lens, num_q_heads=heads[0], num_kv_heads=heads[1], budget=[max_sel * 16 - 5] + [max(0, n // 3 - 20) for n in lens[1:]],
                            p=0.9, heavy_frac=0.01, alpha_range=(0.0, 3.0), shuffle_pool=True, need_v=False, seed=95)
    cache = build_cache(w, bits=bits)
    q, budget = w.q.to(cache.device), w.budget.to(cache.device)
    sa, sb = (T.DecodeStep(cache, max_sel=max_sel, with_kept_idx=True) for _ in range(2))
    sa.select(q, budget)
    sa.prune(q, w.p)
    for again in (False, True):
        for t in (sb.sel_pages, sb.sel_count, sb.kept_count, sb.kept_idx, sb.union_count, sb.union_idx):
            t.fill_(-7)
        T.twilight_prof_enable(1)
        sb.select_prune(None, None, None, q, budget, w.p)
        torch.cuda.synchronize()
        names = [name for name, _ in T.twilight_prof_collect()]
        T.twilight_prof_enable(0)
        assert names == ["page_score", "select_score_topp"]
        _same_lists(sa, sb)


def _random_codes(T, batch, pages, heads, bits=4, pool=4096):
    """Cache of random page bounds and codes (pool pages shared by the sequences), a query."""
    g = torch.Generator(device="cuda").manual_seed(5)
    table = (torch.arange(batch * pages, dtype=torch.int32) * 7 % pool).view(batch, pages)
    cache = T.PagedKV(heads[0], heads[1], table, torch.full((batch,), 16 * pages - 5), pool, need_v=False, quant_bits=bits)
    cache.page_minmax.copy_(torch.randn(pool, heads[1], 2, 128, device="cuda", generator=g).sort(dim=2).values)
    cache.kq_pool.random_(0, 256, generator=g)
    cache.kq_meta[..., 0] = 4.0 / (1 << bits)
    cache.kq_meta[..., 1] = -2.0
    return cache, torch.randn(batch, heads[0], 128, device="cuda", generator=g).to(torch.bfloat16)


@pytest.mark.parametrize("bits,heads,batch,pages,max_sel", [
    (4, (32, 8), 9, 300, 129), (4, (32, 8), 24, 1100, 256), (4, (16, 16), 48, 1024, 200), (8, (16, 8), 40, 2050, 150), (2, (64, 8), 12, 4096, 256),
    (4, (8, 2), 96, 260, 256), (4, (32, 8), 32, 1030, 130), (8, (12, 12), 100, 700, 140), (4, (32, 8), 56, 1024, 129), (2, (32, 8), 56, 1025, 129)])
def test_one_launch_select_prune_of_middling_lists(bits, heads, batch, pages, max_sel):
    """2049 to 4096 candidates on more heads than CUs, three workgroups to a CU (scores in registers) or four (in LDS), by heads and
    table width on both sides of the rule: against the separate calls bit for bit, lists of every length up to the bound."""
    T = _T()
    cache, q = _random_codes(T, batch, pages, heads, bits)
    rng = np.random.default_rng(batch)
    cache.seq_lens[1::2] = torch.from_numpy(rng.integers(0, 16 * pages + 1, batch // 2).astype(np.int32)).cuda()
    budget = torch.from_numpy(rng.integers(0, 16 * max_sel + 100, batch).astype(np.int32)).cuda()
    budget[0] = 16 * max_sel
    sa, sb = (T.DecodeStep(cache, max_sel=max_sel, with_kept_idx=True) for _ in range(2))
    sa.select(q, budget)
    sa.prune(q, 0.9)
    T.twilight_prof_enable(1)
    sb.select_prune(None, None, None, q, budget, 0.9)
    torch.cuda.synchronize()
    names = [name for name, _ in T.twilight_prof_collect()]
    T.twilight_prof_enable(0)
    assert names == ["page_score", "select_score_topp"]
    _same_lists(sa, sb)


def _select_prune_us(T, batch, pages, max_sel):
    """Median time of the one launch that selects, scores and prunes for `batch` x 32 heads."""
    cache, q = _random_codes(T, batch, pages, (32, 8))
    st = T.DecodeStep(cache, max_sel=max_sel)
    budget = torch.full((batch,), 16 * max_sel, dtype=torch.int32, device="cuda")
    for _ in range(3):
        st.select_prune(None, None, None, q, budget, 0.9)
    torch.cuda.synchronize()
    T.twilight_prof_enable(1)
    for _ in range(15):
        st.select_prune(None, None, None, q, budget, 0.9)
    torch.cuda.synchronize()
    us = [ms * 1e3 for name, ms in T.twilight_prof_collect() if name == "select_score_topp"]
    T.twilight_prof_enable(0)
    return float(np.median(us))


def test_two_heads_per_cu_do_not_pay_for_four():
    """512 heads of 3008 candidates take 0.60 of what 1024 do (34.2 and 56.6 us), in the form that puts four to a CU 0.69 (39.0)."""
    T = _T()
    half, full = _select_prune_us(T, 16, 3750, 188), _select_prune_us(T, 32, 3750, 188)
    assert half < 0.645 * full, (half, full)


def _same_lists(sa, sb):
    assert torch.equal(sa.status, sb.status)
    for name, count in (("sel_pages", "sel_count"), ("kept_idx", "kept_count"), ("union_idx", "union_count")):
        ca, cb = getattr(sa, count).flatten().tolist(), getattr(sb, count).flatten().tolist()
        assert ca == cb, name
        xa, xb = (getattr(s, name).reshape(len(ca), -1).cpu() for s in (sa, sb))
        for i, c in enumerate(ca):
            assert torch.equal(xa[i, :c], xb[i, :c]), (name, i)


@pytest.mark.parametrize("G,bits", [(1, 4), (2, 2), (4, 4), (4, 8), (8, 4)])
def test_page_bounds_under_a_long_page_table(G, bits):
    """The bound scores' workgroups cover 32 or 64 pages, by the width of the page table: lists, bounds of every page and
    the cache with the step's token appended are the same under both, at rows that end at the edges of 16-page steps and of workgroups, with unmapped pages, a token on one of them, and a sequence without a new token."""
    T = _T()
    lens = [1, 16 * 32, 16 * 32 + 1, 16 * 64, 16 * 64 + 1, 16 * 128 + 1, 16 * 256, 16 * 256 + 1, 16 * 80 + 5, 16 * 49 - 3, 777]
    w = synth.make_workload("steps", lens, num_q_heads=8 * G, num_kv_heads=8, budget=[max(16, n // 4) for n in lens], p=0.9,
                            heavy_frac=0.01, alpha_range=(0.0, 3.0), shuffle_pool=True, extra_pool_pages=3, seed=29)
    dev = "cuda"
    table = w.page_table.clone()
    table[4, 3] = table[8, 80] = -1                       # (sequence 8: its last page, that of the new token)
    offs = torch.tensor(w.seq_offsets[:-1], dtype=torch.int32, device=dev)
    k, v, q, budget = w.k.to(dev), w.v.to(dev), w.q.to(dev), w.budget.to(dev)
    last = torch.tensor([o - 1 for o in w.seq_offsets[1:]], dtype=torch.int64, device=dev)
    pos = (w.seq_lens.to(dev, torch.int32) - 1).contiguous()
    pos[10] = -1
    max_sel = max(-(-int(b) // 16) for b in w.budget)
    got = []
    for width in (table.shape[1], 3000, 3009):            # 11 x 8 rows: 440 and 4136 workgroups of 64 pages, for 256 CUs
        wide = torch.full((len(lens), width), -1, dtype=torch.int32)
        wide[:, :table.shape[1]] = table
        c = T.PagedKV(8 * G, 8, wide, w.seq_lens, w.num_pool_pages, dev, quant_bits=bits)
        c.append(k, v, torch.zeros_like(pos), torch.where(pos >= 0, c.seq_lens - 1, c.seq_lens), offs, max(lens))
        st = T.DecodeStep(c, max_sel=max_sel)
        st.append_select(k[last].contiguous(), v[last].contiguous(), pos, q, budget)
        torch.cuda.synchronize()
        rows = st.ws_select[:len(lens) * 8 * G * width * 4].view(torch.int32).view(len(lens), 8 * G, width)
        got.append([[rows[b, :, :(n + 15) // 16].cpu() for b, n in enumerate(lens)], c, st])
        again = T.DecodeStep(c, max_sel=max_sel)          # nothing appended: the same lists (sequence 10 has its old bounds either way)
        again.select(q, budget)
        for b in range(len(lens)):
            for h in range(8 * G):
                n = int(st.sel_count[b, h])
                assert n == int(again.sel_count[b, h]) and torch.equal(st.sel_pages[b, h, :n], again.sel_pages[b, h, :n]), (width, b, h)
    base = got[0]
    for rows, c, st in got[1:]:
        for b in range(len(lens)):
            assert torch.equal(rows[b], base[0][b]), (c.max_pages, b)
        for name in ("k_pool", "v_pool", "kq_pool", "kq_meta", "page_minmax"):
            assert torch.equal(getattr(c, name).view(torch.uint8), getattr(base[1], name).view(torch.uint8)), (c.max_pages, name)
    # the bounds themselves, of one sequence, from the cache's page bounds
    mm = base[1].page_minmax[table[7].to(dev).long()].double().cpu()               # [pages, 8, 2, 128]
    qd = w.q[7].double().view(8, G, 1, 128)
    want = torch.maximum(qd * mm[:, :, 0].permute(1, 0, 2)[:, None], qd * mm[:, :, 1].permute(1, 0, 2)[:, None]).sum(-1).view(8 * G, -1)
    have = base[0][7].view(torch.float32).double()
    # 128 fp32 additions: at most 12 in a chain (8 in a lane, 4 levels), each within 2^-24 of sums below the sum of magnitudes
    lim = 12 * 2.0 ** -24 * (qd.abs() * mm.abs().amax(2).permute(1, 0, 2)[:, None]).sum(-1).view(8 * G, -1)
    assert bool(((have - want).abs() <= lim).all())


def _page_score_us(T, batch, max_pages, kv_heads):
    """Median time of the bounds' launch of a step that appends a token, for `batch` ragged sequences of 32 query heads."""
    B = T.binding
    rng = np.random.default_rng(3)
    lens = [int(16 * np.exp(rng.uniform(np.log(max_pages / 32), np.log(max_pages)))) for _ in range(batch)]
    pool = batch * max_pages
    cache = T.PagedKV(32, kv_heads, torch.arange(pool, dtype=torch.int32).view(batch, max_pages), torch.tensor(lens), pool)
    cache.page_minmax.copy_(torch.randn(pool, kv_heads, 2, 128, device="cuda").sort(dim=2).values)
    new = torch.randn(batch, kv_heads, 128, device="cuda").to(torch.bfloat16)
    q = torch.randn(batch, 32, 128, device="cuda").to(torch.bfloat16)
    budget = torch.full((batch,), 256, dtype=torch.int32, device="cuda")
    other = torch.empty(1 << 29, dtype=torch.uint8, device="cuda")          # what a step's other layers leave in the caches
    st = T.DecodeStep(cache, max_sel=16)
    B.twilight_prof_enable(1)
    for _ in range(25):
        other.zero_()
        st.append_select(new, new, cache.seq_lens - 1, q, budget)
    torch.cuda.synchronize()
    us = [ms * 1e3 for name, ms in B.twilight_prof_collect() if name == "page_score"]
    B.twilight_prof_enable(0)
    return float(np.median(us))


@pytest.mark.parametrize("few,many,max_pages,kv_heads", [(124, 128, 256, 8), (126, 130, 19, 32)])
def test_bounds_of_many_short_rows_cost_what_a_few_less_do(few, many, max_pages, kv_heads):
    """Just below and above 4096 workgroups of 64 pages, from where on wide page tables take the form for many pages: it is not for
    rows this short, which took 21.4 us with it against 17.3 (16.8 for the few less) and 15.8 against 12.8."""
    T = _T()
    less, more = _page_score_us(T, few, max_pages, kv_heads), _page_score_us(T, many, max_pages, kv_heads)
    assert more < 1.12 * less, (less, more)


@pytest.mark.parametrize("bits", [2, 4, 8])
def test_token_lists_of_sequences_without_tokens(bits):
    """Lengths of 0 and below next to a sequence of 100 tokens: no entry of an empty sequence's lists lies inside it, whatever
    its value, so its scores are -inf, its integer dot products 0, and nothing of it is kept."""
    T = _T()
    w = synth.make_workload("empty", [100] * 5, num_q_heads=4, num_kv_heads=2, budget=64, p=1.0, seed=97)
    cache = build_cache(w, bits=bits)
    lens = [0, -1, 100, -33, -2 ** 31]
    cache.seq_lens.copy_(torch.tensor(lens, dtype=torch.int32))
    dev, max_cand = cache.device, 272                     # more than the 256 candidates of a scoring workgroup
    ids = np.resize(np.array([-2 ** 31, -4097, -5, -1, 0, 1, 15, 16, 31, 99, 100, 111, 112, 1 << 20, 2 ** 31 - 1], np.int32), max_cand)
    cand = torch.from_numpy(np.tile(ids, (5, 4, 1))).to(dev)
    cnt = torch.tensor([max_cand, 15, 1, 271], dtype=torch.int32, device=dev).repeat(5, 1)
    q = w.q.to(dev)
    sc = torch.full((5, 4, max_cand), 7.0, dtype=torch.float32, device=dev)
    dots = torch.full((5, 4, max_cand, 4), 7, dtype=torch.int32, device=dev)
    T.twilight_int4_score_tokens(cache.kv, q, cand, cnt, max_cand, sc, dots)
    st = T.DecodeStep(cache, max_sel=max_cand // 16, with_kept_idx=True)
    ws = torch.empty(T.twilight_workspace_bytes(T.TW_WS_PRUNE_TOKENS, cache.kv, max_cand), dtype=torch.uint8, device=dev)
    T.twilight_topp_prune_tokens(cache.kv, q, cand, cnt, max_cand, w.p, st.kept_count, st.kept_idx, st.kept_stride,
                                 st.union_count, st.union_idx, st.union_stride, st.status, ws)
    torch.cuda.synchronize()
    for b, n in enumerate(lens):
        for h in range(4):
            c = int(cnt[b, h])
            inside = (ids[:c] >= 0) & (ids[:c] < n)
            assert np.array_equal(np.isfinite(sc[b, h, :c].cpu().numpy()), inside), (b, h)
            assert not dots[b, h, :c].cpu().numpy()[~inside].any(), (b, h)
            assert st.kept_idx[b, h, :int(st.kept_count[b, h])].cpu().numpy().tolist() == ids[:c][inside].tolist(), (b, h)
        for g in range(2):
            inside = np.unique(ids[(ids >= 0) & (ids < n)])
            assert st.union_idx[2 * b + g, :int(st.union_count[2 * b + g])].cpu().numpy().tolist() == inside.tolist(), (b, g)


def _attend_lists(T, G, H, lens, n, seed, bound=0):
    """Attention of sequences of n tokens over lists of lens[l] entries (H lists per sequence), in rows of `bound` entries if the
    longest has no more: outputs against float64.  `combined` of the step returned: whether the lists were cut and combined."""
    batch, P, cols = len(lens) // H, (n + 15) // 16, max(64, int(max(lens)))
    stride = max(cols, bound)
    g = torch.Generator(device="cuda").manual_seed(seed)
    cache = T.PagedKV(G * H, H, torch.randperm(batch * P, generator=torch.Generator().manual_seed(seed)).int().view(batch, P), torch.full((batch,), n), batch * P)
    cache.k_pool.normal_(generator=g)
    cache.v_pool.normal_(generator=g)
    q = torch.randn(batch, G * H, 128, device="cuda", generator=g).to(torch.bfloat16)
    lens = torch.as_tensor(lens, device="cuda")
    idx = torch.rand(len(lens), n, device="cuda", generator=g).argsort(dim=1)[:, :cols]
    idx = idx.masked_fill(torch.arange(idx.shape[1], device="cuda") >= lens[:, None], n).sort(dim=1).values       # n: does not count
    st = T.DecodeStep(cache, max_sel=1, union_stride=stride)
    st.union_count.copy_(lens)
    st.union_idx.fill_(-1)
    st.union_idx[:, :idx.shape[1]].copy_(idx)
    torch.cuda.synchronize()
    T.twilight_prof_enable(1)
    st.attend(q)
    torch.cuda.synchronize()
    st.combined = [name for name, _ in T.twilight_prof_collect()] == ["sparse_decode", "combine"]
    T.twilight_prof_enable(0)
    page = cache.page_table.long().gather(1, idx.clamp(max=n - 1).view(batch, -1) // 16).view(len(lens), -1)
    head = (torch.arange(len(lens), device="cuda") % H)[:, None]
    for lo in range(0, len(lens), 64):
        s = slice(lo, lo + 64)
        k, v = (pool[page[s], head[s], idx[s] % 16].double() for pool in (cache.k_pool, cache.v_pool))
        live = (idx[s] < n)[:, None, :]
        logit = ((q.view(len(lens), G, 128)[s].double()[:, :, None] * k[:, None]).sum(-1) / 128 ** 0.5).masked_fill(~live, float("-inf"))
        m = logit.amax(-1, keepdim=True).clamp(min=-1e300)
        w = (logit - m).exp()
        want = (w[..., None] * v[:, None]).sum(2) / w.sum(-1, keepdim=True).clamp(min=1e-300)
        out = st.out.view(len(lens), G, 128)[s].double()
        # bf16 result (2^-9 of a value), fp32 logits of bf16 products: the bars of the other attention tests
        assert bool(((out - want).norm(dim=-1) <= 4e-3 * want.norm(dim=-1) + 1e-6).all()), lo
        lse = (m + w.sum(-1, keepdim=True).log()).squeeze(-1)
        have = st.lse.view(len(lens), G)[s].double()
        empty = ~live.any(-1).expand_as(have)
        assert bool(torch.isneginf(have[empty]).all()) and bool(((have - lse).abs()[~empty] <= 1e-3 * lse.abs()[~empty].clamp(min=1.0)).all()), lo
    return st


@pytest.mark.parametrize("bound", [0, 1344], ids=["narrow_rows", "wide_rows"])
@pytest.mark.parametrize("G,lists,longest,kind", [
    (1, 72, 180, "same"), (2, 256, 300, "mixed"), (4, 512, 129, "same"), (8, 520, 946, "same"), (4, 744, 377, "mixed"), (1, 1088, 745, "mixed"),
    (2, 1280, 500, "same"), (8, 1384, 200, "mixed"), (1, 2048, 900, "same"), (1, 6144, 40, "mixed"), (2, 776, 64, "empty")])
def test_attention_over_many_lists(G, lists, longest, kind, bound):
    """More than 64 lists, one, two and more to a thread of the item map: equal ones (whole or in equal pieces), lists of
    widely different lengths, of which many are shorter than a chunk, and mostly empty ones, against float64.  In rows of 1344
    entries; in rows as wide as the longest list those short enough take a workgroup each and no item map."""
    T = _T()
    rng = np.random.default_rng(lists)
    lens = np.full(lists, longest)
    if kind != "same":
        lens = np.exp(rng.uniform(0, np.log(longest + 1), lists)).astype(np.int64)
        lens[rng.integers(lists)] = longest
    if kind == "empty":
        lens[rng.random(lists) < 0.9] = 0
    st = _attend_lists(T, G, 8, lens, 2 * longest, seed=lists + G, bound=bound)
    assert st.combined or not bound


@pytest.mark.parametrize("lists,longest,chunk", [(256, 300, 128), (128, 300, 128), (256, 220, 64), (120, 300, 64)])
def test_middling_lists_of_single_heads_are_cut_into_two_steps(lists, longest, chunk):
    """One query head per KV head: items of 128 entries for at least 128 lists of at least 144 entries on average (in items
    of 64 256 lists of 160 took 11.8 us instead of 10.9), of 64 below; lists of 20 entries up to the longest, in rows so wide that
    lists are cut."""
    T = _T()
    lens = np.linspace(20, longest, lists).astype(np.int64)
    assert (lens.mean() >= 144) == (longest == 300)
    st = _attend_lists(T, 1, 8, lens, 2 * longest, seed=lists, bound=1344)
    first = st.ws_decode[:4 * (lists + 1)].view(torch.int32).cpu().numpy()
    assert np.array_equal(np.diff(first), -(-lens // chunk))


@pytest.mark.parametrize("G,lists,bound", [(1, 64, 512), (1, 136, 768), (1, 1376, 768), (2, 64, 512), (4, 64, 512), (8, 64, 256), (2, 136, 768), (4, 264, 768), (8, 136, 512), (8, 264, 512)])
def test_short_lists_take_a_workgroup_each_up_to_the_line(G, lists, bound):
    """At the bound up to which a workgroup takes a list whole (2 * lists below and above the 256 CUs, lists above them) and one entry
    beyond it, where lists are cut: a list as long as its row, some a step or two long, empty ones, against float64."""
    T = _T()
    for width, cut in ((bound, False), (bound + 1, True)):
        lens = np.resize([width, 0, width // 16, 64, 65, 128, 129, 1], lists)
        st = _attend_lists(T, G, 8, lens, 2 * bound, seed=lists + bound)
        assert st.combined == cut and T.twilight_decode_whole(st.cache.kv, T.TW_WS_DECODE, width) != cut, width


@pytest.mark.parametrize("bound,items,chunk", [(512, 6, None), (2048, 12, 64)])
def test_balance_of_the_work_list_of_lists_taken_whole(bound, items, chunk):
    """The benchmark's report on lists that are not cut, which leave nothing in the workspace, and on the same ones cut."""
    import bench
    T = _T()
    st = _attend_lists(T, 2, 3, np.array([128, 64, 130, 1, 64, 200]), 400, seed=1, bound=bound)
    if chunk is None:
        st.ws_decode.fill_(255)
    got = bench.decode_balance(T, st.cache, st)
    assert got["items"] == items and got["chunk"] == chunk
    if chunk is None:
        assert got["grid_workgroups"] == 6 and got["rows_per_workgroup_max_over_mean"] == pytest.approx(200 * 6 / 587)


@pytest.mark.parametrize("G,lists,bound", [(1, 128, 1280), (4, 136, 1280), (4, 264, 1280), (8, 136, 768), (8, 136, 1280), (8, 264, 1280)])
def test_a_long_list_among_short_ones_is_shared_out(G, lists, bound):
    """One list as long as its row among ones a sixteenth of it costs what it does in rows of 4096 entries, where lists are cut: taken
    whole by a workgroup it was 18 to 35 us of attention instead of 11 to 18."""
    T = _T()
    B, lens, us = T.binding, np.full(lists, bound // 16), []
    lens[lists // 3] = bound
    for width in (bound, 4096):
        st = _attend_lists(T, G, 8, lens, 2 * bound, seed=lists, bound=width)
        q = torch.randn(lists // 8, 8 * G, 128, device="cuda").to(torch.bfloat16)
        B.twilight_prof_enable(1)
        for _ in range(24):
            st.attend(q)
        torch.cuda.synchronize()
        kern = {}
        for name, ms in B.twilight_prof_collect():
            kern.setdefault(name, []).append(ms * 1e3)
        B.twilight_prof_enable(0)
        us.append(sum(float(np.median(v)) for v in kern.values()))
    assert us[0] < 1.1 * us[1], us


def _dense_us(T, batch, n):
    """Median time of dense attention over `batch` sequences of n tokens, 2 query heads on each of 8 KV heads."""
    B = T.binding
    P = (n + 15) // 16
    cache = T.PagedKV(16, 8, torch.arange(batch * P, dtype=torch.int32).view(batch, P), torch.full((batch,), n), batch * P)
    q = torch.randn(batch, 16, 128, device="cuda").to(torch.bfloat16)
    st = T.DecodeStep(cache, max_sel=1)
    for _ in range(3):
        st.dense(q)
    torch.cuda.synchronize()
    B.twilight_prof_enable(1)
    for _ in range(15):
        st.dense(q)
    torch.cuda.synchronize()
    us = [ms * 1e3 for name, ms in B.twilight_prof_collect() if name == "sparse_decode"]
    B.twilight_prof_enable(0)
    return float(np.median(us))


def test_lists_about_as_many_as_workgroups_are_shared_evenly():
    """560 lists of 1440 tokens cost what 280 of 2880 do (65.4 and 68.0 us): cut into a long and a short piece each, with the
    long pieces all on the same workgroups, they took 85.5."""
    T = _T()
    many, few = _dense_us(T, 70, 1440), _dense_us(T, 35, 2880)
    assert many < 1.12 * few, (many, few)


def _range_ends(heads, scale=1.0):
    """Queries whose int8 values are at the ends of their range and of its 4-bit halves, against keys whose codes are 0 and 15 in
    whole groups."""
    Hq, Hkv = heads
    ramp = np.concatenate([np.arange(-127, -63), np.arange(64, 128)])
    rows = [np.full(128, 127), np.full(128, -127), np.where(np.arange(128) % 2, 127, -127), ramp, np.roll(ramp[::-1], 5),
            np.resize([-16, -1, 15, 16, 112, 119, 120, 127], 128), np.resize([0, -128 + 1, 8, -8, 7, -9], 128), np.arange(128)]
    n = 40
    w = synth.make_workload("ends", [n] * len(rows), num_q_heads=Hq, num_kv_heads=Hkv, budget=32, p=0.9, need_v=False, seed=97)
    for b, row in enumerate(rows):
        w.q[b] = torch.from_numpy(np.stack([np.roll(row, 7 * h) for h in range(Hq)]).astype(np.float32) * scale).to(torch.bfloat16)
    w.k[::3] = torch.where(torch.arange(128) % 2 == 0, 1.0, -1.0).to(torch.bfloat16)       # codes 15 and 0
    w.k[1::5, :, :64] = 2.0                                                                   # constant groups
    return w, n


def _range_ends_want(w, b, h):
    """The oracle's integer dots and scores of a head over its sequence's tokens."""
    u, s, z = O.quantize_k(synth.bits(w.seq_k(b)[:, h // (w.num_q_heads // w.num_kv_heads)]))
    qi, sq = O.quantize_q(synth.bits(w.q[b, h]))
    return O.int4_dots(qi, u)[0], O.int4_scores(qi, sq, u, s, z)


@pytest.mark.parametrize("heads", [(2, 2), (4, 2)])
def test_dots_at_the_ends_of_the_query_and_code_ranges(heads):
    """Integer dots of 4-bit codes bit for bit where the query's int8 values are at the ends of their range and of its 4-bit
    halves, against keys whose codes are 0 and 15 in whole groups."""
    T = _T()
    Hq, Hkv = heads
    w, n = _range_ends(heads)
    cache = build_cache(w)
    stride = cache.page_table.shape[1] * 16
    sc = torch.zeros(w.batch, Hq, stride, dtype=torch.float32, device="cuda")
    dots = torch.zeros(w.batch, Hq, stride, 4, dtype=torch.int32, device="cuda")
    T.twilight_int4_score(cache.kv, w.q.cuda(), None, None, 0, sc, dots)
    torch.cuda.synchronize()
    for b in range(w.batch):
        for h in range(Hq):
            I, S = _range_ends_want(w, b, h)
            assert np.array_equal(dots[b, h, :n].cpu().numpy(), I), (b, h)
            assert np.array_equal(sc[b, h, :n].cpu().numpy(), S), (b, h)


@pytest.mark.parametrize("heads", [(2, 2), (4, 2), (4, 1)])
@pytest.mark.parametrize("tokens", [False, True], ids=["pages", "tokens"])
def test_dots_of_lists_at_the_ends_of_the_query_and_code_ranges(heads, tokens):
    """The same through the scoring of page lists and of token lists."""
    T = _T()
    Hq, Hkv = heads
    w, n = _range_ends(heads)
    cache = build_cache(w)
    item = 1 if tokens else 16
    entries = list(range(n)) if tokens else [0, 2, 1]
    order = np.concatenate([np.arange(e * item, min(n, (e + 1) * item)) for e in entries])           # the slots' tokens ...
    slots = np.concatenate([np.arange(i * item, i * item + min(n, (e + 1) * item) - e * item) for i, e in enumerate(entries)])
    length = 48 if tokens else 3
    lists = torch.zeros(w.batch, Hq, length, dtype=torch.int32, device="cuda")
    lists[..., :len(entries)] = torch.tensor(entries, dtype=torch.int32, device="cuda")
    count = torch.full((w.batch, Hq), len(entries), dtype=torch.int32, device="cuda")
    sc = torch.zeros(w.batch, Hq, 48, dtype=torch.float32, device="cuda")
    dots = torch.zeros(w.batch, Hq, 48, 4, dtype=torch.int32, device="cuda")
    score = T.twilight_int4_score_tokens if tokens else T.twilight_int4_score
    score(cache.kv, w.q.cuda(), lists, count, length, sc, dots)
    torch.cuda.synchronize()
    for b in range(w.batch):
        for h in range(Hq):
            I, S = _range_ends_want(w, b, h)
            assert np.array_equal(dots[b, h].cpu().numpy()[slots], I[order]), (b, h)
            assert np.array_equal(sc[b, h].cpu().numpy()[slots], S[order]), (b, h)


@pytest.mark.parametrize("heads,max_sel", [((2, 2), 3), ((4, 1), 3), ((4, 2), 200), ((4, 1), 500)])
def test_kept_sets_at_the_ends_of_the_query_and_code_ranges(heads, max_sel):
    """The same scores inside the one-launch selector + pruner, by the tokens that it keeps (the query scaled by a power of
    two, which leaves its integers alone and spreads the weights over the tokens)."""
    T = _T()
    w, n = _range_ends(heads, scale=2.0 ** -8)
    cache = build_cache(w)
    st = T.DecodeStep(cache, max_sel=max_sel, with_kept_idx=True)
    for p in (0.3, 0.9, 0.99):
        st.select_prune(None, None, None, w.q.cuda(), torch.full((w.batch,), n, dtype=torch.int32, device="cuda"), p)
        torch.cuda.synchronize()
        for b in range(w.batch):
            for h in range(heads[0]):
                S = _range_ends_want(w, b, h)[1]
                mask, tau = O.topp_set(S, float(np.float32(p)))                  # (p crosses the C ABI as a float)
                got = np.isin(np.arange(n), st.kept_idx[b, h, :int(st.kept_count[b, h])].cpu().numpy())
                W = O.softmax_weights(S)
                assert np.all(np.abs(W[got != mask] - tau) <= 1e-6), (b, h, p)


@pytest.mark.parametrize("pages,take", [(8192, 8191), (16384, 8191), (16384, 8192), (16384, 8193), (32768, 8192), (32768, 8193), (32700, 31)])
def test_page_lists_of_the_longest_rows(pages, take):
    """Lists of about 8192 entries and a short one, of rows at and just under the selection kernels' longest."""
    T = _T()
    lens = [16 * pages, 16 * (pages - 100)]
    cache, q = _random_bounds(T, lens, pages, heads=(2, 1), pool=4096, seed=pages + take)
    st = T.DecodeStep(cache, max_sel=take)
    st.select(q, torch.full((2,), 16 * take, dtype=torch.int32, device="cuda"))
    torch.cuda.synchronize()
    mm = cache.page_minmax.cpu()
    for b, n in enumerate(lens):
        rows = mm[cache.page_table[b, :n // 16].cpu().long(), 0]
        for h in range(2):
            U = O.page_upper_bounds(synth.bits(q[b, h].cpu()), u16(rows[:, 0]), u16(rows[:, 1]))
            want = O.select_pages(U, 16 * take, n)
            assert st.sel_pages[b, h, :int(st.sel_count[b, h])].cpu().numpy().tolist() == want.tolist(), (b, h)


def _infinite_bounds(T, P, seqs, high, low, seed):
    """Cache of `seqs` sequences of P pages of which `high` have an infinite bound, `low` minus infinity and one the largest
    and one the smallest finite bound (their difference is infinite too); a query of positive values."""
    g = torch.Generator().manual_seed(seed)
    cache = T.PagedKV(2, 1, torch.arange(P, dtype=torch.int32).view(1, P).repeat(seqs, 1), torch.tensor([16 * P] * seqs), P, need_v=False)
    mm = torch.randn(P, 1, 2, 128, generator=g).sort(dim=2).values
    at = torch.randperm(P, generator=g)
    mm[at[:high]], mm[at[high:high + low]] = 3e38, -3e38
    for page, sign in ((at[-1], 1.0), (at[-2], -1.0)):
        mm[page], mm[page, :, :, 0] = 0.0, sign * 3e38
    cache.page_minmax.copy_(mm.to(torch.bfloat16))
    q = torch.randn(seqs, 2, 128, generator=g).abs() + 1e-3
    q[:, :, 0] = 1.0
    return cache, q.to(torch.bfloat16)


def _infinite_bounds_want(cache, q, P, take):
    mm = cache.page_minmax.cpu()
    with np.errstate(over="ignore"):
        return [O.select_pages(O.page_upper_bounds(synth.bits(q[b, h]), u16(mm[:, 0, 0]), u16(mm[:, 0, 1])), 16 * take, 16 * P).tolist()
                for b in range(q.shape[0]) for h in range(2)]


@pytest.mark.parametrize("high,low", [(0, 0), (1, 0), (0, 1), (3, 5), (90, 100)])
@pytest.mark.parametrize("P", [400, 600, 2050, 8194, 16388, 32768])
def test_page_lists_of_rows_with_infinite_bounds(P, high, low):
    """Bounds that overflow, and finite ones whose difference does, in rows of every selection kernel: the threshold among the
    finite bounds, among the infinite ones and below them."""
    T = _T()
    cache, q = _infinite_bounds(T, P, 1, high, low, P + high)
    for take in sorted({1, 70, P // 3, P - 60, P - 1}):
        st = T.DecodeStep(cache, max_sel=take)
        st.select(q.cuda(), torch.full((1,), 16 * take, dtype=torch.int32, device="cuda"))
        torch.cuda.synchronize()
        got = [st.sel_pages[0, h, :int(st.sel_count[0, h])].cpu().numpy().tolist() for h in range(2)]
        assert got == _infinite_bounds_want(cache, q, P, take), take


@pytest.mark.parametrize("P,seqs,take", [(400, 1, 50), (400, 200, 50), (2000, 1, 100), (4000, 1, 200), (4000, 200, 200), (4000, 200, 400), (8192, 2, 300)])
def test_one_launch_selection_of_rows_with_infinite_bounds(P, seqs, take):
    """The same where the pages are picked inside the pruner's kernel."""
    T = _T()
    for high, low in ((0, 0), (5, 3), (take + 40, 70)):
        cache, q = _infinite_bounds(T, P, seqs, high, low, P + take)
        st = T.DecodeStep(cache, max_sel=take)
        st.select_prune(None, None, None, q.cuda(), torch.full((seqs,), 16 * take, dtype=torch.int32, device="cuda"), 0.9)
        torch.cuda.synchronize()
        got = [r[:n].tolist() for r, n in zip(st.sel_pages.view(2 * seqs, -1).cpu().numpy(), st.sel_count.view(-1).cpu().numpy())]
        assert got == _infinite_bounds_want(cache, q, P, take), (high, low)
