// Stage 1: Quest-style page selector (paper: Section 4.1 "Token Selector",
// Section 4 challenge C1: pooling per 16-token page).
//
// page_score:  U[h,P] = sum_d max(q_d*min[P,d], q_d*max[P,d]).  16 lanes per
//              page, each lane one 16-byte load of min and of max (8 dims);
//              the G query heads of the KV head share the loaded bounds.
//              fp32 order: 8 dims left to right per lane, then a pairwise
//              DPP tree over the 16 lanes (bit-reproducible).
// page_select: per (sequence, query head) the Kp largest bounds, ties to the
//              lower page id, ascending: rows of up to 32768 entries in
//              registers (select_body.h), longer ones by a 4 x 8-bit radix
//              select on the order-preserving key over global memory.
//
// page_score with APPEND also appends the decode step's one new token per sequence on its way
// (twilight_append_select): the 16 lanes that own the page the token falls into store its K/V
// rows, quantise K, and fold it into the page's bounds before scoring them.
#include <atomic>
#include <stdlib.h>
#include "tw_common.h"
#include "kquant_common.h"
#include "topp_common.h"
#include "select_body.h"

namespace {

constexpr int PS_PAGES_PER_WG = 32;   // 4 waves x 4 pages x 2 iterations
constexpr int PS_LONG_PAGES = 64;     // of a workgroup of the form for many pages: 4 iterations

struct ScoreArgs {
  const uint32_t* q;          // bf16 pairs [b][Hq][64]
  const uint4* page_minmax;   // [page][Hkv][2][16]
  const int32_t* page_table;
  const int32_t* seq_lens;
  float* scores;              // [b][Hq][max_pages]
  int Hq, Hkv, max_pages;
  long long pool_pages;
  // the step's new token (APPEND only): one row per sequence, [b][Hkv][128] bf16
  const uint4* k_new;
  const uint4* v_new;         // or nullptr
  const int32_t* new_pos;     // [b] position of the new token, < 0: none
  uint4* k_pool;              // or nullptr (no bf16 copy kept)
  uint4* v_pool;
  uint32_t* kq_pool;          // INT4 codes, 16 words per token
  uint32_t* kq_meta;
  uint4* page_minmax_w;
  uint32_t* arrive;           // [b][Hkv] arrival counters of a top-p launch that follows, cleared here, or nullptr
  const int32_t* budget;      // with ORDER: the sequences' budgets ...
  int batch, max_sel;         // ... their number, and the bound of the lists
};

// The sequences in the order of their heads' work in a launch that follows, the most first: place i's at tw_order_word(i).  By one
// workgroup, a sequence a thread.  (A listed page's scores cost about what sixteen pages' bounds do.)
__device__ __forceinline__ void ps_order(const ScoreArgs& a) {
  static_assert(TW_ORDER_MAX <= 256, "a thread a sequence");
  const int tid = threadIdx.x, lane = tid & 63;
  auto work = [&](int i) -> int {
    if (i >= a.batch) return -1;
    int P, K;
    tw_select_sizes<TW_PAGE>(a.seq_lens[i], a.budget[i], a.max_pages, a.max_sel, &P, &K);
    return K * 16 + P;
  };
  const int mine = work(tid);
  int rank = 0;
  for (int i0 = 0; i0 < a.batch; i0 += 64) {
    const int other = work(i0 + lane);
#pragma unroll 8
    for (int j = 0; j < 64; ++j) {
      const int w = __builtin_amdgcn_readlane(other, j);
      rank += w > mine || (w == mine && i0 + j < tid) ? 1 : 0;
    }
  }
  if (tid < a.batch) a.arrive[tw_order_word(rank, a.Hkv)] = (uint32_t)tid;
}

// The step's new token, by the 16 lanes that own its page: its K/V rows stored, K quantised, the page's bounds (*rmn, *rmx)
// folded and stored.
template <int BITS>
__device__ __forceinline__ void ps_append(const ScoreArgs& a, long long row, long long page, int g, int sp, int seg, uint4* rmn, uint4* rmx) {
  const uint4 raw = a.k_new[row * 16 + seg];
  const long long slot = (page * a.Hkv + g) * TW_PAGE + (sp & 15);
  if (a.k_pool) a.k_pool[slot * 16 + seg] = raw;
  if (a.v_new) a.v_pool[slot * 16 + seg] = a.v_new[row * 16 + seg];
  float x[8];
  tw_unpack8(raw, x);
  uint32_t word, word2, meta;
  tw_quantize_lane8<BITS>(x, seg, &word, &word2, &meta);
  if (BITS == 4) a.kq_pool[slot * 16 + seg] = word;
  else if (BITS == 8) ((uint2*)a.kq_pool)[slot * 16 + seg] = make_uint2(word, word2);
  else if ((seg & 1) == 0) a.kq_pool[slot * 8 + (seg >> 1)] = word;
  if ((seg & 3) == 0) a.kq_meta[slot * 4 + (seg >> 2)] = meta;
  // bounds: the token alone if it opens the page, else folded into the page's older tokens
  float mn[8], mx[8];
  tw_unpack8(*rmn, mn);
  tw_unpack8(*rmx, mx);
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    mn[i] = (sp & 15) ? fminf(mn[i], x[i]) : x[i];
    mx[i] = (sp & 15) ? fmaxf(mx[i], x[i]) : x[i];
  }
  // min / max of bf16 values are bf16 values: the top 16 bits are exact
  uint4 wmn, wmx;
  wmn.x = (__float_as_uint(mn[0]) >> 16) | (__float_as_uint(mn[1]) & 0xFFFF0000u);
  wmn.y = (__float_as_uint(mn[2]) >> 16) | (__float_as_uint(mn[3]) & 0xFFFF0000u);
  wmn.z = (__float_as_uint(mn[4]) >> 16) | (__float_as_uint(mn[5]) & 0xFFFF0000u);
  wmn.w = (__float_as_uint(mn[6]) >> 16) | (__float_as_uint(mn[7]) & 0xFFFF0000u);
  wmx.x = (__float_as_uint(mx[0]) >> 16) | (__float_as_uint(mx[1]) & 0xFFFF0000u);
  wmx.y = (__float_as_uint(mx[2]) >> 16) | (__float_as_uint(mx[3]) & 0xFFFF0000u);
  wmx.z = (__float_as_uint(mx[4]) >> 16) | (__float_as_uint(mx[5]) & 0xFFFF0000u);
  wmx.w = (__float_as_uint(mx[6]) >> 16) | (__float_as_uint(mx[7]) & 0xFFFF0000u);
  uint4* pm = a.page_minmax_w + (page * a.Hkv + g) * 32;
  pm[seg] = wmn;
  pm[16 + seg] = wmx;
  *rmn = wmn;
  *rmx = wmx;
}

// The bounds of a page for the G heads, by its 16 lanes; put(h, bound) in the lane that ends with head h's.
// (The signs of 4 heads' queries fill the scalar registers; those of further heads are compared anew, or they spill.  With 8 heads
//  and the append page_score_long_kernel still spills 8 scalar registers, page_score_kernel none; the variants that leave the order of
//  work spill more: 15 with 8 heads and 3 with 4, both with the append, on long tables, 2 to 5 with 8 heads on short ones.)
template <int G, typename Put>
__device__ __forceinline__ void ps_score(float (&q)[G][8], const uint4& cmn, const uint4& cmx, int seg, Put put) {
  float mn[8], mx[8];
  tw_unpack8(cmn, mn);
  tw_unpack8(cmx, mx);
  float part[G];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    float acc = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      // the product of two bf16 values is exact in fp32, so this fused
      // multiply-add rounds exactly like "acc + q*v"
      if (h >= 4) asm volatile("" : "+v"(q[h][i]));
      const float v = q[h][i] > 0.f ? mx[i] : mn[i];
      acc = __builtin_fmaf(q[h][i], v, acc);
    }
    part[h] = acc;
  }
  if constexpr (G >= 4) {
    // The pairwise tree over the 16 lanes (l^1, l^2, l^4, l^8) for four heads at once: at the first two levels a
    // lane keeps the half of its values that one bit of its lane id selects and adds the partner's copy of them
    // (the same two operands as the plain tree adds, so the same sums), which leaves lane l with the quad sum of
    // head 2 * (l & 1) + ((l >> 1) & 1); the last two levels rotate the row by 4 and by 8 (a lane reads lane
    // l - 4, then l - 8, modulo 16), which for lanes 4..7 are exactly l ^ 4 and l ^ 8 of the same head.  Lanes 4..7
    // end with the four totals: 5 additions and 6 selects per four heads instead of 16 additions.
    const bool b0 = seg & 1, b1 = seg & 2;
#pragma unroll
    for (int h4 = 0; h4 < G; h4 += 4) {
      const float k0 = b0 ? part[h4 + 2] : part[h4 + 0], s0 = b0 ? part[h4 + 0] : part[h4 + 2];
      const float k1 = b0 ? part[h4 + 3] : part[h4 + 1], s1 = b0 ? part[h4 + 1] : part[h4 + 3];
      const float a0 = __fadd_rn(k0, tw_dpp_f<TW_DPP_XOR1>(s0));     // head h4 + 2 * b0
      const float a1 = __fadd_rn(k1, tw_dpp_f<TW_DPP_XOR1>(s1));     // head h4 + 2 * b0 + 1
      const float kk = b1 ? a1 : a0, ss = b1 ? a0 : a1;
      float t = __fadd_rn(kk, tw_dpp_f<TW_DPP_XOR2>(ss));            // head h4 + 2 * b0 + b1, summed over the quad
      t = __fadd_rn(t, tw_dpp_f<0x124>(t));                          // row_ror:4 - lanes 4..7 and 12..15 read l ^ 4
      t = __fadd_rn(t, tw_dpp_f<0x128>(t));                          // row_ror:8 - every lane reads l ^ 8
      if ((seg >> 2) == 1)
        put(h4 + 2 * (seg & 1) + ((seg >> 1) & 1), __fadd_rn(t, 0.0f));
    }
  } else {
#pragma unroll
    for (int h = 0; h < G; ++h) {
      const float acc = tw_row16_sum(part[h]);
      if (seg == 0) put(h, __fadd_rn(acc, 0.0f));
    }
  }
}

template <int G, bool APPEND, int BITS = 4, bool ORDER = false>
__global__ __launch_bounds__(256) void page_score_kernel(ScoreArgs a) {
  // KV head fastest in dispatch order: the 8 heads' bounds of a pool page are 4 KiB contiguous,
  // and the workgroups that read them start next to each other
  const int b = blockIdx.z, g = blockIdx.x;
  const int tid = threadIdx.x, seg = tid & 15, grp = tid >> 4;   // grp: 0..15 page slot in the WG
  TW_STAMP(0);
  const int n = a.seq_lens[b];
  const int pos_early = APPEND && ORDER ? a.new_pos[b] : -1;       // (with the stores of ps_order behind it not a scalar load any more further down)
  // last pages first: the workgroup that appends the step's new token (the sequence's last page) has the longest
  // chain of dependent accesses and should not be the one that starts last
  const int base = (int)(gridDim.y - 1 - blockIdx.y) * PS_PAGES_PER_WG;
  // page-table entries of this lane's 4 pages: issued before the sequence length is known (any entry of
  // the row may be read; entries beyond the last page are ignored below), so that the two loads overlap
  constexpr int IT = PS_PAGES_PER_WG / 16;
  long long pool[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int lp = base + it * 16 + grp;
    pool[it] = a.page_table[(long long)b * a.max_pages + (lp < a.max_pages ? lp : a.max_pages - 1)];
  }
  int P = (n + TW_PAGE - 1) / TW_PAGE;
  if (P > a.max_pages) P = a.max_pages;
  // (the counters of a top-p launch that follows are cleared on the way out, after every load of the kernel: a store
  //  ahead of them would turn the scalar loads of the prologue into vector loads that wait for one another)
  const bool clears = a.arrive && blockIdx.y == 0 && tid <= G;      // the group's counter and one per head
  const bool orders = ORDER && base == 0 && (blockIdx.x | blockIdx.z) == 0;    // (does not leave early, whatever that sequence's length)
  if (base >= P && !orders) {
    if (clears) a.arrive[(b * a.Hkv + g) * TW_CTR + tid] = 0;
    return;
  }

  // q of the G heads, the 8 dims of this lane; the sign decides which corner
  // of the [min,max] box maximises q_d * k_d.
  float q[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const uint4 r = *(const uint4*)(a.q + ((long long)(b * a.Hq + g * G + h)) * 64 + seg * 4);
    tw_unpack8(r, q[h]);
  }

  // then all 8 bound loads (clamped addresses, unconditional) so that they are in flight together;
  // unmapped pages are masked afterwards
  bool live[IT], ok[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) live[it] = base + it * 16 + grp < P;
  uint4 rmn[IT], rmx[IT];
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    ok[it] = live[it] && pool[it] >= 0 && pool[it] < a.pool_pages;
    const uint4* pm = a.page_minmax + ((ok[it] ? pool[it] : 0) * a.Hkv + g) * 32;
    rmn[it] = tw_ld_stream(pm + seg);
    rmx[it] = tw_ld_stream(pm + 16 + seg);
  }
  if (APPEND) {
    // the page of the new token, if it lies in this workgroup's pages: its 16 owner lanes append
    const int sp = ORDER ? pos_early : a.new_pos[b];
    const int off = (sp >> 4) - base;
    if (sp >= 0 && sp < n && off >= 0 && off < PS_PAGES_PER_WG && (off & 15) == grp) {
#pragma unroll
      for (int it = 0; it < IT; ++it) {
        if (it == (off >> 4) && ok[it]) {
          ps_append<BITS>(a, (long long)b * a.Hkv + g, pool[it], g, sp, seg, &rmn[it], &rmx[it]);
        }
      }
    }
  }
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const int lp = base + it * 16 + grp;
    ps_score<G>(q, rmn[it], rmx[it], seg, [&](int h, float t) {
      if (live[it])
        a.scores[((long long)(b * a.Hq + g * G + h)) * a.max_pages + lp] = ok[it] ? t : -3.402823466e38f;   // unmapped page: ranks last
    });
  }
  if (clears) a.arrive[(b * a.Hkv + g) * TW_CTR + tid] = 0;
  if constexpr (ORDER) { if (orders) ps_order(a); }
}

// The same for many pages.  What bounds page_score_kernel there is that a workgroup waits for its length, then its page-table
// entries, then two steps' bounds, and ends; its scores are pieces of 16 bytes.  Here a workgroup asks for four steps' bounds at
// once (at most 128 registers, four workgroups per CU), its page-table entries are one load per wave, the new token comes
// last, where the registers are free, and the scores leave through LDS in whole lines.  Decode steps, us: 16 x 32768 tokens,
// 64 heads over 8 127.1 -> 123.9, 32 x 32768, 32 over 8 144.5 -> 142.3, 64 ragged sequences of up to 65536 241.8 -> 233.8.
template <int G, bool APPEND, int BITS = 4, bool ORDER = false>
__global__ __launch_bounds__(256, 4) void page_score_long_kernel(ScoreArgs a) {
  constexpr int STEPS = PS_LONG_PAGES / 16;
  // KV head fastest in dispatch order: the 8 heads' bounds of a pool page are 4 KiB contiguous,
  // and the workgroups that read them start next to each other
  const int b = blockIdx.z, g = blockIdx.x;
  const int tid = threadIdx.x, lane = tid & 63, seg = tid & 15, grp = tid >> 4;   // grp: 0..15 page slot in a step
  __shared__ float sh[G][PS_LONG_PAGES], sh_app[G];
  TW_STAMP(0);
  const int n = a.seq_lens[b];
  // last pages first: the workgroup that appends the step's new token (the sequence's last page) has the longest
  // chain of dependent accesses and should not be the one that starts last
  const int base = (int)(gridDim.y - 1 - blockIdx.y) * PS_LONG_PAGES;
  // all page-table entries of the wave's pages in one load, lane 4 * it + j that of page j of step it: issued before the
  // sequence length is known (any entry of the row may be read; entries beyond the last page are ignored below)
  const int mine = base + ((lane >> 2) < STEPS ? lane >> 2 : 0) * 16 + (tid >> 6) * 4 + (lane & 3);
  int entry = a.page_table[(long long)b * a.max_pages + (mine < a.max_pages ? mine : a.max_pages - 1)];
  int P = (n + TW_PAGE - 1) / TW_PAGE;
  if (P > a.max_pages) P = a.max_pages;
  // (the counters of a top-p launch that follows are cleared on the way out, after every load of the kernel: a store
  //  ahead of them would turn the scalar loads of the prologue into vector loads that wait for one another)
  const bool clears = a.arrive && blockIdx.y == 0 && tid <= G;      // the group's counter and one per head
  const bool orders = ORDER && base == 0 && (blockIdx.x | blockIdx.z) == 0;    // (does not leave early, whatever that sequence's length)
  if (base >= P && !orders) {
    if (clears) a.arrive[(b * a.Hkv + g) * TW_CTR + tid] = 0;
    return;
  }
  const int pages = P - base < PS_LONG_PAGES ? P - base : PS_LONG_PAGES, steps = (pages + 15) >> 4;

  // q of the G heads, the 8 dims of this lane; the sign decides which corner
  // of the [min,max] box maximises q_d * k_d.
  float q[G][8];
#pragma unroll
  for (int h = 0; h < G; ++h) {
    const uint4 r = *(const uint4*)(a.q + ((long long)(b * a.Hq + g * G + h)) * 64 + seg * 4);
    tw_unpack8(r, q[h]);
  }
  // the page of the new token, if it lies in this workgroup's pages
  int app = -1, sp = 0;
  if (APPEND) {
    sp = a.new_pos[b];
    const int off = (sp >> 4) - base;
    if (sp >= 0 && sp < n && off >= 0 && off < PS_LONG_PAGES) app = off;
  }
  if (mine >= P || entry < 0 || entry >= a.pool_pages) entry = -1;

  // clamped addresses, unconditional loads, so that they are in flight together and their waits can be counted;
  // unmapped pages and steps beyond the last are masked afterwards
  int pool[STEPS];
  uint4 rmn[STEPS], rmx[STEPS];
#pragma unroll
  for (int it = 0; it < STEPS; ++it) {
    pool[it] = __shfl(entry, it * 4 + (lane >> 4), 64);
    const uint4* pm = a.page_minmax + ((long long)(pool[it] >= 0 ? pool[it] : 0) * a.Hkv + g) * 32;
    rmn[it] = tw_ld_stream(pm + seg);
    rmx[it] = tw_ld_stream(pm + 16 + seg);
  }
#pragma unroll
  for (int it = 0; it < STEPS; ++it) {
    if (it >= steps) break;                       // (block-uniform)
    // unmapped page: ranks last
    ps_score<G>(q, rmn[it], rmx[it], seg, [&](int h, float t) { sh[h][it * 16 + grp] = pool[it] >= 0 ? t : -3.402823466e38f; });
  }
  // The new token, behind the steps, where the registers are free: one row of lanes of the wave that has its page.  (The steps
  // saw the page's old bounds: its scores are kept apart.)
  if (APPEND && app >= 0 && (tid >> 6) == ((app & 15) >> 2)) {                      // (wave-uniform)
    const int page = __shfl(entry, (app >> 4) * 4 + (app & 3), 64);
    if (page < 0) {
      if (lane < G) sh_app[lane] = -3.402823466e38f;
    } else if (lane < 16) {
      const uint4* pm = a.page_minmax + ((long long)page * a.Hkv + g) * 32;
      uint4 mn = pm[seg], mx = pm[16 + seg];
      ps_append<BITS>(a, (long long)b * a.Hkv + g, page, g, sp, seg, &mn, &mx);
      ps_score<G>(q, mn, mx, seg, [&](int h, float t) { sh_app[h] = t; });
    }
  }
  __syncthreads();
#pragma unroll
  for (int i = tid; i < G * PS_LONG_PAGES; i += 256) {
    const int h = i / PS_LONG_PAGES, j = i % PS_LONG_PAGES;
    if (j < pages) a.scores[((long long)(b * a.Hq + g * G + h)) * a.max_pages + base + j] = j == app ? sh_app[h] : sh[h][j];
  }
  if (clears) a.arrive[(b * a.Hkv + g) * TW_CTR + tid] = 0;
  if constexpr (ORDER) { if (orders) ps_order(a); }
}

struct SelectArgs {
  const float* scores;        // [b][Hq][max_pages]
  const int32_t* seq_lens;
  const int32_t* budget;
  int32_t* sel_pages;         // [b][Hq][max_sel]
  int32_t* sel_count;
  int Hq, max_pages, max_sel;
  int p_above, p_upto;        // the register kernel takes the heads with p_above < pages <= p_upto
};
// The kernels' UNIT parameter = tokens per row entry: 16 = pages (budget and lengths are in tokens), 1 = the rows hold one
// score per token (channel-sparse token selector; max_pages is then the row length in tokens).

template <int UNIT>
__device__ __forceinline__ void tw_select_sizes(const SelectArgs& a, int n, int B, int* P_out, int* K_out) {
  ::tw_select_sizes<UNIT>(n, B, a.max_pages, a.max_sel, P_out, K_out);
}

template <int UNIT>
__global__ __launch_bounds__(256) void page_select_kernel(SelectArgs a) {
  const int b = blockIdx.y, h = blockIdx.x, tid = threadIdx.x;
  int P, Kp;
  tw_select_sizes<UNIT>(a, a.seq_lens[b], a.budget[b], &P, &Kp);
  const float* sc = a.scores + ((long long)(b * a.Hq + h)) * a.max_pages;
  int32_t* out = a.sel_pages + ((long long)(b * a.Hq + h)) * a.max_sel;
  if (tid == 0) a.sel_count[b * a.Hq + h] = Kp;
  if (Kp == 0) return;
  if (Kp == P) {                         // budget covers the sequence: every page
    for (int i = tid; i < P; i += 256) out[i] = i;
    return;
  }

  __shared__ uint32_t hist[256];
  __shared__ uint32_t wsum[17];
  __shared__ uint32_t sh_prefix, sh_remaining;
  uint32_t prefix = 0, remaining = (uint32_t)Kp;
  // radix select of the Kp-th largest key, 8 bits per pass from the top
#pragma unroll 1
  for (int shift = 24; shift >= 0; shift -= 8) {
    hist[tid] = 0;
    __syncthreads();
    const uint32_t himask = shift == 24 ? 0u : (0xFFFFFFFFu << (shift + 8));
    for (int i = tid; i < P; i += 256) {
      const uint32_t key = tw_float_key(sc[i]);
      if ((key & himask) == prefix) atomicAdd(&hist[(key >> shift) & 255u], 1u);
    }
    __syncthreads();
    // thread t looks at digit 255-t: inclusive count of keys with digit >= its own
    const uint32_t mine = hist[255 - tid];
    uint32_t total;
    const uint32_t incl = tw_block_scan_u32(mine, wsum, &total);
    if (incl >= remaining && incl - mine < remaining) {
      sh_prefix = prefix | ((uint32_t)(255 - tid) << shift);
      sh_remaining = remaining - (incl - mine);
    }
    __syncthreads();
    prefix = sh_prefix;
    remaining = sh_remaining;
    __syncthreads();
  }
  // prefix = key of the Kp-th largest bound; `remaining` pages with exactly
  // that key are taken, lowest ids first.
  const uint32_t T = prefix, need_eq = remaining;
  uint32_t run_gt = 0, run_eq = 0;
#pragma unroll 1
  for (int base = 0; base < P; base += 256) {
    const int i = base + tid;
    uint32_t key = 0;
    const bool in = i < P;
    if (in) key = tw_float_key(sc[i]);
    const uint32_t fgt = (in && key > T) ? 1u : 0u;
    const uint32_t feq = (in && key == T) ? 1u : 0u;
    uint32_t total;
    const uint32_t incl = tw_block_scan_u32(fgt | (feq << 16), wsum, &total);
    const uint32_t gt_before = run_gt + (incl & 0xFFFFu) - fgt;
    const uint32_t eq_before = run_eq + (incl >> 16) - feq;
    if (fgt || (feq && eq_before < need_eq)) {
      const uint32_t pos = gt_before + (eq_before < need_eq ? eq_before : need_eq);
      if (pos < (uint32_t)a.max_sel) out[pos] = i;
    }
    run_gt += total & 0xFFFFu;
    run_eq += total >> 16;
  }
}


// The body of page_select_reg_kernel for a row of at most NT * E entries of which 0 < Kp < P are taken.  reach: slots that
// are looked at, P or, with more than 8 slots per thread, whose keys say where the row ends, anything above.
template <int NT, int E, int SNB>
__device__ __forceinline__ void select_row(const float* sc, int P, int reach, int Kp, int max_sel, int32_t* out, uint32_t* hist,
                                           unsigned long long* cand, uint32_t* cnt) {
  const int tid = threadIdx.x;
  uint32_t key[E], T, need_eq;
#pragma unroll
  for (int e = 0; e < E; ++e) {                   // clamped loads, all in flight
    const int i = e * NT + tid;
    key[e] = __float_as_uint(sc[i < P ? i : P - 1]);
  }
#pragma unroll
  for (int e = 0; e < E; ++e)
    key[e] = E > 8 ? tw_select_key(__uint_as_float(key[e]), e * NT + tid < P) : tw_float_key(__uint_as_float(key[e]));
  tw_select_threshold<NT, E, SNB, 10>(key, reach, (uint32_t)Kp, hist, cand, &T, &need_eq);
  tw_select_list<NT, E>(key, reach, T, need_eq, cnt, [&](uint32_t pos, int e) {
    if (pos < (uint32_t)max_sel) out[pos] = e * NT + tid;
  });
}

// Rows of at most NT * E entries, the keys in registers.
// 8 and 16 slots per thread (rows of 2049 to 16384 entries): what bounds many rows is how many workgroups wait at their
// barriers side by side, so these forms are held to 64 registers - two workgroups of 16 waves per CU - with 512 buckets, 8
// per scanning lane.  1024 rows x 2500 entries 27.9 us with 72 registers and 1024 buckets, one workgroup per CU -> 21.3,
// x 8192 37.9 -> 29.5 (256 x 8192, a row per CU: 8.9 as before); 1024 rows x 16384 in the 32-slot form 78 -> 42.
// Above 8 slots a row of up to a quarter of the form's length takes a body of its own, with fewer slots and without the
// longest rows' sentinel keys: 64 ragged sequences x 32 heads of up to 32768 tokens 105 -> 78 us, up to 9000 37.9 -> 31.5.
// The longest rows, which reach every group of slots, take one without the groups' branches (256 x 32768 27.9 -> 27.7; without it the
// others compile the worse, 512 x 20000 tokens 26.3 -> 27.4).
// A list's entries are stored as they are found: gathered in LDS and sent off in whole lines they take one barrier more and gain nothing
// (256 x 4096 of 32768 entries 27.8 us stored, 28.0 gathered, 256 x 4096 of 32768 tokens 21.9 and 22.3, 32 x 312 of 2500 5.8 and 6.1).
template <int NT, int E, int UNIT>
__global__ __launch_bounds__(NT, E == 8 || E == 16 ? 8 : 1) void page_select_reg_kernel(SelectArgs a) {
  constexpr int SNB = E > 16 ? 2048 : (NT == 1024 && E == 2 ? 1024 : 512);
  const int b = blockIdx.y, h = blockIdx.x, tid = threadIdx.x;
  int P, Kp;
  tw_select_sizes<UNIT>(a, a.seq_lens[b], a.budget[b], &P, &Kp);
  if (P <= a.p_above || P > a.p_upto) return;     // another launch's head (block-uniform)
  int32_t* out = a.sel_pages + ((long long)(b * a.Hq + h)) * a.max_sel;
  const float* sc = a.scores + ((long long)(b * a.Hq + h)) * a.max_pages;
  if (tid == 0) a.sel_count[b * a.Hq + h] = Kp;
  if (Kp == 0) return;
  if (Kp == P) {
    for (int i = tid; i < P; i += NT) out[i] = i;
    return;
  }
  __shared__ __align__(16) uint32_t hist[tw_sel_words(SNB)];
  __shared__ unsigned long long cand[SEL_CAP];
  __shared__ uint32_t cnt[E * NT / 64];
  constexpr int SHORT = E > 16 ? 8 : 4;
  if (E > 8 && P <= SHORT * NT) select_row<NT, SHORT, 512>(sc, P, P, Kp, a.max_sel, out, hist, cand, cnt);   // (block-uniform)
  else if (E > 16 && P > (E - SEL_GROUP) * NT) {
    int n = P;
    asm volatile("" : "+s"(n));                   // (nothing in common with the next body: what the compiler shared it spilled)
    select_row<NT, E, SNB>(sc, n, E * NT, Kp, a.max_sel, out, hist, cand, cnt);
  }
  else select_row<NT, E, SNB>(sc, P, P, Kp, a.max_sel, out, hist, cand, cnt);
}

template <int G, bool ORDER>
void launch_score(const ScoreArgs& a, dim3 grid, bool many, bool append, int bits, hipStream_t s) {
  if (many) {
    if (!append)        TW_LAUNCH((page_score_long_kernel<G, false, 4, ORDER>), grid, dim3(256), 0, s, a);
    else if (bits == 4) TW_LAUNCH((page_score_long_kernel<G, true, 4, ORDER>), grid, dim3(256), 0, s, a);
    else if (bits == 8) TW_LAUNCH((page_score_long_kernel<G, true, 8, ORDER>), grid, dim3(256), 0, s, a);
    else                TW_LAUNCH((page_score_long_kernel<G, true, 2, ORDER>), grid, dim3(256), 0, s, a);
  }
  else if (!append)   TW_LAUNCH((page_score_kernel<G, false, 4, ORDER>), grid, dim3(256), 0, s, a);
  else if (bits == 4) TW_LAUNCH((page_score_kernel<G, true, 4, ORDER>), grid, dim3(256), 0, s, a);
  else if (bits == 8) TW_LAUNCH((page_score_kernel<G, true, 8, ORDER>), grid, dim3(256), 0, s, a);
  else                TW_LAUNCH((page_score_kernel<G, true, 2, ORDER>), grid, dim3(256), 0, s, a);
}
template <int G>
void launch_score(const ScoreArgs& a, dim3 grid, bool many, bool order, bool append, int bits, hipStream_t s) {
  if (order) launch_score<G, true>(a, grid, many, append, bits, s);
  else launch_score<G, false>(a, grid, many, append, bits, s);
}

}  // namespace

#ifdef TW_PHASE_TIMING
extern "C" int twilight_debug_stamps_select(unsigned long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(tw_dbg_stamps), sizeof(unsigned long long) * 64) == hipSuccess ? 0 : -1;
}
#endif

// The selection kernels by row length (entries per row = sa.max_pages) and number of heads.
template <int UNIT>
static int launch_select(SelectArgs sa, const TwDims& d, hipStream_t s) {
  const int L = sa.max_pages;
  sa.p_above = -1; sa.p_upto = L;
  const dim3 grid(d.Hq, d.batch);
  // Many heads and rows of up to 8192 entries (ragged batches): rows of at most 2048 entries go to a 256-thread launch
  // of their own, eight of which share a CU (two of the 1024-thread kernel).
  if (L > 2048 && L <= SEL_REG_PAGES && (long long)d.batch * d.Hq > 2ll * tw_num_cus()) {
    sa.p_upto = 2048;
    tw_prof_before(TW_K_PAGE_SELECT, s);
    TW_LAUNCH((page_select_reg_kernel<256, 8, UNIT>), grid, dim3(256), 0, s, sa);
    if (int e = tw_prof_after(s)) return e;
    sa.p_above = 2048; sa.p_upto = L;
  }
  tw_prof_before(TW_K_PAGE_SELECT, s);
  // rows of 513..2048 entries: with few heads (at most two workgroups per CU) the 1024-thread variant is the
  // quicker one (6.7 against 8.4 us at 8 x 32 heads x 2048 pages); many heads are better served by small workgroups
  const bool few_heads = (long long)d.batch * d.Hq <= 2ll * tw_num_cus();
  if (L <= 512)
    TW_LAUNCH((page_select_reg_kernel<256, 2, UNIT>), grid, dim3(256), 0, s, sa);
  else if (L <= 2048 && !few_heads)
    TW_LAUNCH((page_select_reg_kernel<256, 8, UNIT>), grid, dim3(256), 0, s, sa);
  else if (L <= 2048)
    TW_LAUNCH((page_select_reg_kernel<1024, 2, UNIT>), grid, dim3(1024), 0, s, sa);
  else if (L <= SEL_REG_PAGES)
    TW_LAUNCH((page_select_reg_kernel<1024, 8, UNIT>), grid, dim3(1024), 0, s, sa);
  else if (L <= SEL_REG_TWO)
    TW_LAUNCH((page_select_reg_kernel<1024, 16, UNIT>), grid, dim3(1024), 0, s, sa);
  else if (L <= SEL_REG_MAX)
    TW_LAUNCH((page_select_reg_kernel<1024, 32, UNIT>), grid, dim3(1024), 0, s, sa);
  else
    TW_LAUNCH(page_select_kernel<UNIT>, grid, dim3(256), 0, s, sa);
  return tw_prof_after(s);
}

// page_score_long_kernel from 16 of its workgroups per CU on, on page tables of at least 1536 pages (one query head per KV head:
// 512).  Steps in both forms, us: 16 x 32768 tokens (4096 workgroups) 86.3 / 85.1, 32 ragged sequences of up to 32768 76.7 / 75.3,
// 48 of up to 24576 87.3 / 85.5; with fewer workgroups it does not fill the chip (512: 2 x 32768 36.2 / 37.2).  On narrower tables
// a workgroup in a few has the new token, whose bounds and quantised row come last in its chain, and a ragged batch's rows fill few
// of its 64 pages: 128 ragged of up to 4096 75.6 / 78.7, of up to 8192 91.7 / 93.3, 32 of up to 16384 49.6 / 50.7 (full rows of
// 16384 gain, 64 x 16384 154.2 / 151.8, but their lengths are not known here).  With one query head the rest of the chain is
// shorter: the kernel alone, 32 KV heads, 128 ragged of up to 8192 67.7 / 63.7, of up to 2048 22.9 / 22.3, of up to 1024 16.1 / 17.2,
// 192 x 300 17.5 / 21.5; 16 KV heads, 64 of up to 4096 12.5 / 14.0.  128 pages per workgroup: 64 ragged of up to 16384 86.4 / 88.6.
static int score_columns(const TwDims& d) { return (d.max_pages + PS_LONG_PAGES - 1) / PS_LONG_PAGES; }
static bool score_many(const TwDims& d) {
  return (long long)d.batch * d.Hkv * score_columns(d) >= 16ll * tw_num_cus() && d.max_pages >= (d.G == 1 ? 512 : 1536);
}

static int select_impl(const twilight_kv_t* kv, const void* q, const int32_t* budget_tokens,
                       int32_t* sel_pages, int32_t* sel_count, int32_t max_sel,
                       void* ws, size_t ws_bytes, void* stream,
                       bool append, const void* k_new, const void* v_new, const int32_t* new_pos,
                       uint32_t* arrive = nullptr, bool bounds_only = false, bool order = false) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !budget_tokens || !sel_pages || !sel_count || max_sel <= 0 || !kv->page_minmax) return TW_EINVAL;
  if (append) {
    if (!k_new || !new_pos || !kv->kq_pool || !kv->kq_meta) return TW_EINVAL;
    if (v_new && !kv->v_pool) return TW_EINVAL;
  }
  if (!ws || ws_bytes < twilight_workspace_bytes(TW_WS_SELECT, kv, max_sel, 0)) return TW_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;

  ScoreArgs a;
  a.q = (const uint32_t*)q; a.page_minmax = (const uint4*)kv->page_minmax;
  a.page_table = kv->page_table; a.seq_lens = kv->seq_lens; a.scores = (float*)ws;
  a.Hq = d.Hq; a.Hkv = d.Hkv; a.max_pages = d.max_pages; a.pool_pages = d.pool_pages;
  a.k_new = (const uint4*)k_new; a.v_new = (const uint4*)v_new; a.new_pos = new_pos;
  a.k_pool = (uint4*)kv->k_pool; a.v_pool = (uint4*)kv->v_pool;
  a.kq_pool = (uint32_t*)kv->kq_pool; a.kq_meta = (uint32_t*)kv->kq_meta;
  a.page_minmax_w = (uint4*)kv->page_minmax;
  a.arrive = arrive;
  a.budget = budget_tokens; a.batch = d.batch; a.max_sel = max_sel;
  const bool many = score_many(d);
  const dim3 grid(d.Hkv, many ? score_columns(d) : (d.max_pages + PS_PAGES_PER_WG - 1) / PS_PAGES_PER_WG, d.batch);
  tw_prof_before(TW_K_PAGE_SCORE, s);
  switch (d.G) {
    case 1: launch_score<1>(a, grid, many, order, append, d.bits, s); break;
    case 2: launch_score<2>(a, grid, many, order, append, d.bits, s); break;
    case 4: launch_score<4>(a, grid, many, order, append, d.bits, s); break;
    default: launch_score<8>(a, grid, many, order, append, d.bits, s); break;
  }
  if (int e = tw_prof_after(s)) return e;
  if (bounds_only) return TW_OK;

  SelectArgs sa;
  sa.scores = (const float*)ws; sa.seq_lens = kv->seq_lens; sa.budget = budget_tokens;
  sa.sel_pages = sel_pages; sa.sel_count = sel_count;
  sa.Hq = d.Hq; sa.max_pages = d.max_pages; sa.max_sel = max_sel;
  return launch_select<TW_PAGE>(sa, d, s);
}

// Channel-sparse token selector (a Double-Sparsity-style base algorithm in front of the pruner; Section 4.1's
// black-box token selector, Sections 4.3 / 5): every token of a sequence is scored from the INT4 copy of K with the
// query restricted to the KV head's channel set, and the budget's worth of tokens with the largest estimate is handed
// over as a token list (ties to the lower position, ascending).
extern "C" int twilight_ds_select_tokens(const twilight_kv_t* kv, const void* q, const uint32_t* channel_mask,
                                         const int32_t* budget_tokens, int32_t* cand_tokens, int32_t* cand_count,
                                         int32_t max_cand, void* ws, size_t ws_bytes, void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !channel_mask || !budget_tokens || !cand_tokens || !cand_count || max_cand <= 0 || !kv->kq_pool || !kv->kq_meta)
    return TW_EINVAL;
  if ((long long)d.max_pages * TW_PAGE > 0x7FFFFFFFll / 4) return TW_EINVAL;
  if (!ws || ws_bytes < twilight_workspace_bytes(TW_WS_DS_SELECT, kv, max_cand, 0)) return TW_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  if (int e = tw_score_all_tokens_masked(kv, d, q, channel_mask, (float*)ws, s)) return e;
  SelectArgs sa;
  sa.scores = (const float*)ws; sa.seq_lens = kv->seq_lens; sa.budget = budget_tokens;
  sa.sel_pages = cand_tokens; sa.sel_count = cand_count;
  sa.Hq = d.Hq; sa.max_pages = d.max_pages * TW_PAGE; sa.max_sel = max_cand;
  return launch_select<1>(sa, d, s);
}

extern "C" int twilight_select_pages(const twilight_kv_t* kv, const void* q, const int32_t* budget_tokens,
                                     int32_t* sel_pages, int32_t* sel_count, int32_t max_sel,
                                     void* ws, size_t ws_bytes, void* stream) {
  return select_impl(kv, q, budget_tokens, sel_pages, sel_count, max_sel, ws, ws_bytes, stream, false, nullptr, nullptr, nullptr);
}

// ---- the selector for callers that must not allocate: same kernels, the bound scores go to a
// fixed array of device memory that the library's code object carries.  The array's name is only a
// host-side handle; its address on the current device comes from hipGetSymbolAddress, once per device.
static __device__ __align__(256) unsigned char scratch[TW_STATIC_SELECT_WS_BYTES];

static int static_scratch_ptr(void** out) {
  static std::atomic<void*> ptrs[TW_MAX_DEVICES];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= TW_MAX_DEVICES) return TW_ELAUNCH;
  void* p = ptrs[dev].load(std::memory_order_acquire);
  if (!p) {
    // every GPU holds its own copy of the array at its own address; racing first calls look up the same value
    if (hipGetSymbolAddress(&p, HIP_SYMBOL(scratch)) != hipSuccess || !p) {
      (void)hipGetLastError();
      return TW_ELAUNCH;
    }
    ptrs[dev].store(p, std::memory_order_release);
  }
  *out = p;
  return TW_OK;
}

extern "C" int twilight_select_pages_static(const twilight_kv_t* kv, const void* q, const int32_t* budget_tokens,
                                            int32_t* sel_pages, int32_t* sel_count, int32_t max_sel, void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (max_sel <= 0) return TW_EINVAL;
  const size_t need = twilight_workspace_bytes(TW_WS_SELECT, kv, max_sel, 0);
  if (need == 0) return TW_EINVAL;
  if (need > (size_t)TW_STATIC_SELECT_WS_BYTES) return TW_ELIMIT;
  void* ws = nullptr;
  if (int e = static_scratch_ptr(&ws)) return e;
  // every score the select kernels read is written by page_score in this call: nothing has to start at zero
  return select_impl(kv, q, budget_tokens, sel_pages, sel_count, max_sel, ws, need, stream, false, nullptr, nullptr, nullptr);
}

extern "C" int twilight_append_select(const twilight_kv_t* kv, const void* k_new, const void* v_new, const int32_t* new_pos,
                                      const void* q, const int32_t* budget_tokens,
                                      int32_t* sel_pages, int32_t* sel_count, int32_t max_sel,
                                      void* ws, size_t ws_bytes, void* stream) {
  return select_impl(kv, q, budget_tokens, sel_pages, sel_count, max_sel, ws, ws_bytes, stream, true, k_new, v_new, new_pos);
}

// Selector and pruner in one call (Section 4.1's pipeline up to the pruned index sets): page bounds (with the step's
// new token appended on the way when k_new is given), then - where the lists are short enough for a workgroup's
// registers - a single launch that picks each head's pages, scores their tokens from the quantised copy of K, runs top-p and
// builds the group's union; otherwise the launches of twilight_select_pages and twilight_topp_prune.
extern "C" int twilight_select_prune(const twilight_kv_t* kv, const void* k_new, const void* v_new, const int32_t* new_pos,
                                     const void* q, const int32_t* budget_tokens, float p,
                                     int32_t* sel_pages, int32_t* sel_count, int32_t max_sel,
                                     int32_t* kept_count, int32_t* kept_idx, int32_t kept_stride,
                                     int32_t* union_count, int32_t* union_idx, int32_t union_stride,
                                     uint32_t* status, void* ws, size_t ws_bytes, void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !budget_tokens || !sel_pages || !sel_count || !kept_count || !union_count || !union_idx || !status ||
      !kv->kq_pool || !kv->kq_meta || max_sel <= 0) return TW_EINVAL;
  if (!(p > 0.f) || p > 1.f || union_stride <= 0 || (kept_idx && kept_stride <= 0)) return TW_EINVAL;
  if ((long long)max_sel * TW_PAGE > (1ll << 22)) return TW_EINVAL;
  const size_t sel_bytes = twilight_workspace_bytes(TW_WS_SELECT, kv, max_sel, 0);
  const size_t need = twilight_workspace_bytes(TW_WS_SELECT_PRUNE, kv, max_sel, 0);
  if (!ws || need == 0 || ws_bytes < need) return TW_EWORKSPACE;
  void* ws_prune = (char*)ws + sel_bytes;
  const bool append = k_new != nullptr;
  // 2: selection and scoring inside the top-p kernel, 1: scoring only, 0: the separate launches
  const int can = tw_prune_fused_ok(d, max_sel, true) ? 2 : (tw_prune_fused_ok(d, max_sel, false) ? 1 : 0);
  int mode = can;
  // fewer heads than CUs with long lists: one workgroup per head cannot pull its list fast enough (32 heads x 8192
  // candidates: 51.8 us per step separately, 56.0 us fused); several per head can, the scoring launch's many too
  if (max_sel * TW_PAGE > 4096 && (long long)d.batch * d.Hq < tw_num_cus()) mode = 0;
  const int parts = tw_prune_parts(d, max_sel);
  if (parts > 1) mode = 2;
#ifdef TW_TUNING
  if (const char* e = getenv("TW_FUSE")) { const int m = atoi(e); mode = parts > 1 ? mode : (m < can ? m : can); }
#endif
  if (mode == 0) {
    if (int e = select_impl(kv, q, budget_tokens, sel_pages, sel_count, max_sel, ws, sel_bytes, stream, append, k_new, v_new,
                            new_pos)) return e;
    return twilight_topp_prune(kv, q, sel_pages, sel_count, max_sel, p, kept_count, kept_idx, kept_stride, union_count,
                               union_idx, union_stride, status, ws_prune, ws_bytes - sel_bytes, stream);
  }
  uint32_t* arrive = (uint32_t*)((char*)ws_prune + tw_prune_layout(d, max_sel, false).arrive);
  // Sequences whose heads' work differs, in more workgroups than run at once: the most first (ps_order), or what begins last ends long
  // after the rest.  Steps, us, as they come / in order: 64 ragged sequences of up to 65536 tokens 222.8 / 206.6, 40 161.2 / 143.8, 16 with
  // 64 heads 92.0 / 84.7, 32 of up to 32768 69.9 / 65.3, 48 of up to 20000 with an eighth in the lists 81.3 / 78.1, with a quarter
  // 90.4 / 84.4.  With shorter lists heads differ less, and the order costs 0.4 us of bounds and a load ahead of all others in every
  // workgroup: 64 ragged of up to 20000 with an eighth in the lists, of 8-bit codes 94.0 / 95.4 (of 2-bit codes 88.7 / 87.7), 128 of up to
  // 8192 87.5 / 88.1, 64 x 12000 129.5 / 129.9.
  const bool order = mode == 2 && parts == 1 && max_sel * TW_PAGE > 2560 && d.batch > 1 && d.batch <= TW_ORDER_MAX &&
                     (long long)d.batch * d.Hq > 3ll * tw_num_cus();
  if (int e = select_impl(kv, q, budget_tokens, sel_pages, sel_count, max_sel, ws, sel_bytes, stream, append, k_new, v_new,
                          new_pos, arrive, mode == 2, order)) return e;
  return tw_prune_fused(kv, d, q, mode == 2 ? (const float*)ws : nullptr, budget_tokens, sel_pages, sel_count, max_sel, p,
                        kept_count, kept_idx, kept_stride, union_count, union_idx, union_stride, status, ws_prune,
                        parts, order, (hipStream_t)stream);
}
