// Stage 3: variable-budget sparse decode attention over the paged bf16 KV
// cache (paper: Definition 3.1 restricted to the kept set and renormalised
// over it; Appendix B.2: every query head of a KV head attends over the
// group's union, the group-wise variable-length form; Section 4.2 load balancing: the
// (sequence, KV head) lists are flattened into equal-sized work items).
//
// Work item = (list, chunk of `chunk` consecutive list entries).  Every wave reads the lists' lengths, derives the
// chunk length that gives each workgroup of the grid the same number of rows (decode_chunk) and finds its
// workgroup's item by a prefix sum over its lanes, so no host round trip and no extra launch is needed.  Inside an
// item the four waves walk their rows without meeting: 16 lanes own one token row (a 16-byte load of K and of V each,
// 8 dims), the G query heads of the group share every loaded row, and each wave keeps its own online-softmax state;
// the states are merged by log-sum-exp, first the workgroup's, then those of a list's items by the combine kernel.
//
// The same kernel serves the per-head variant (the head-wise form of Appendix
// B.2): one list per query head, G = 1, list l reads KV head l / group size.
#include <stdlib.h>
#include <atomic>
#include "tw_common.h"

namespace {

constexpr float kLog2eRsqrtD = 0x1.0527dcp-3f;   // fp32(log2(e) / sqrt(128))
constexpr float kLn2 = 0x1.62e43p-1f;
constexpr float kNegBig = -1.0e30f;              // finite stand-in for -inf in running maxima
constexpr unsigned DEC_MAX_ROUNDS = 3;           // items per workgroup that decode_chunk weighs against each other
constexpr unsigned DEC_UNIT = 64;                // entries of a step of the four waves
constexpr unsigned DEC_ITEM_ROWS = 64;           // rows that an item's set-up and merge are worth ...
constexpr unsigned DEC_CUT_ROWS = 64;            // ... and that merging the pieces of cut lists is

struct DecodeArgs {
  const uint4* q;             // bf16 [b][Hq][16 x uint4]
  const uint4* k_pool;        // 16 uint4 per token row
  const uint4* v_pool;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const int32_t* union_count; // or nullptr (dense)
  const int32_t* union_idx;   // or nullptr (dense)
  uint4* out;                 // bf16 [b][Hq][16 x uint4]
  float* lse;                 // or nullptr
  int32_t* ws_prefix;         // [NG + 1]
  float2* ws_ml;              // [items][G]
  float2* ws_acc;             // [items][G][64 x float2]
  int Hq, Hkv, max_pages, union_stride, NG;
  int chunk0;                 // shortest chunk
  int LH, kv_div;             // lists per sequence (Hkv, or Hq with one list per query head); list l reads KV head l / kv_div
  long long pool_pages;
};

__device__ __forceinline__ float tw_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

template <int K>
__device__ __forceinline__ int tw_row_bcast_i(int v) { return __builtin_amdgcn_update_dpp(0, v, 0x150 + K, 0xF, 0xF, false); }
// row_newbcast:k - lane k of each row of 16 to all lanes of the row
template <int K>
__device__ __forceinline__ float tw_row_bcast(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x150 + K, 0xF, 0xF, false));
}
#define TW_DPP_ROR4 0x124
#define TW_DPP_ROR8 0x128

typedef __bf16 tw_bf16x2 __attribute__((ext_vector_type(2)));
// a.lo * b.lo + a.hi * b.hi + c on bf16 pairs (v_dot2c_f32_bf16)
__device__ __forceinline__ float tw_dot2_bf16(uint32_t a, uint32_t b, float c) {
  return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(tw_bf16x2, a), __builtin_bit_cast(tw_bf16x2, b), c, false);
}

// v_permlane16_swap / v_permlane32_swap: x and y exchange odd with even rows of 16 lanes, or upper with lower halves
__device__ __forceinline__ void tw_swap16(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void tw_swap32(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]); y = __uint_as_float(r[1]);
}
// over the wave's four rows of 16 lanes, every lane gets the result
__device__ __forceinline__ float tw_rows_max(float x) {
  float y = x;
  tw_swap16(x, y); x = fmaxf(x, y); y = x;
  tw_swap32(x, y);
  return fmaxf(x, y);
}
__device__ __forceinline__ float tw_rows_sum(float x) {
  float y = x;
  tw_swap16(x, y); x += y; y = x;
  tw_swap32(x, y);
  return x + y;
}

// Chunk length for T list entries in NG lists on W workgroups: r items per workgroup, with the r whose rows and items'
// fixed cost are least; a list's last chunk is taken to be half full.  The workgroups then end together.  (Chunks of 64,
// 128 or 256 entries, whichever left at most three items to a workgroup, had 1230 items on 1024 workgroups at 8 x 32768
// tokens: 12.6 us against 11.8.  Chunks of any multiple of 16 entries leave a wave's last step partly empty: 1.7 us more
// with one query head per KV head, whose rows need the fewest instructions.)
__device__ __forceinline__ uint32_t decode_chunk(uint32_t T, uint32_t NG, uint32_t W, uint32_t chunk0, uint32_t* rounds) {
  uint32_t best = 0xFFFFFFFFu, chunk = chunk0;
  const uint32_t r0 = 1u + NG / W;                 // (every list is an item)
  *rounds = r0;
#pragma unroll
  for (uint32_t k = 0; k < DEC_MAX_ROUNDS; ++k) {
    uint32_t c = (T / (W * (r0 + k) - NG / 2u) + DEC_UNIT) & ~(DEC_UNIT - 1u);
    c = c < chunk0 ? chunk0 : c;
    const uint32_t cost = (r0 + k) * (c + DEC_ITEM_ROWS);
    if (cost < best) { best = cost; chunk = c; *rounds = r0 + k; }
  }
  return chunk;
}
// more than that many items after all (lists whose last chunks are emptier)
__device__ __forceinline__ uint32_t decode_longer(uint32_t chunk) { return chunk + (((chunk >> 5) + DEC_UNIT) & ~(DEC_UNIT - 1u)); }

// The same for more than 64 lists, where whole lists can be the better items.  Lane j of the wave weighs one way, 0 .. 3: every
// list in at most j + 1 pieces, which is certain to leave a workgroup no more than ceil(NG * (j + 1) / W) items; 4 .. 6: the
// three of decode_chunk, which may turn out more (many short lists: their last chunks are emptier).
struct DecodePlan {
  uint32_t W, chunk, rounds;   // the best of the ways and its items per workgroup
  uint32_t other;              // chunk of the best of the other numbers of items, 0: none
  uint32_t longer, best, best_chunk;
  int state;
  __device__ __forceinline__ DecodePlan(uint32_t T, uint32_t longest, uint32_t NG, uint32_t W_, uint32_t chunk0) : W(W_), state(0) {
    const uint32_t lane = threadIdx.x & 63u, k = lane < 4u ? lane + 1u : 1u;
    const bool sure = lane < 4u;
    const uint32_t units = (longest + DEC_UNIT - 1u) / DEC_UNIT;
    const uint32_t q = (sure ? NG * k + W - 1u : NG) / W, r = sure ? q : q + lane - 3u;
    const uint32_t len = (sure ? units + k - 1u : T) / (sure ? k : W * r - NG / 2u);
    uint32_t c = sure ? len * DEC_UNIT : (len + DEC_UNIT) & ~(DEC_UNIT - 1u);
    c = c < chunk0 ? chunk0 : c;
    const bool whole = c >= units * DEC_UNIT;
    const uint32_t cost = lane < 4u + DEC_MAX_ROUNDS ? r * ((whole ? units * DEC_UNIT : c) + DEC_ITEM_ROWS) + (whole ? 0u : DEC_CUT_ROWS) : 0xFFFFFFFFu;
    // of equals the first: fewer items
    auto least = [&](uint32_t x) -> int { return __builtin_ctzll(__ballot(x == ~tw_wave_max_u32(~x))); };
    const int at = least(cost), at_sure = least(sure ? cost : 0xFFFFFFFFu);
    chunk = longer = (uint32_t)__builtin_amdgcn_readlane((int)c, at);
    rounds = (uint32_t)__builtin_amdgcn_readlane((int)r, at);
    best = (uint32_t)__builtin_amdgcn_readlane((int)cost, at_sure);
    best_chunk = (uint32_t)__builtin_amdgcn_readlane((int)c, at_sure);
    const uint32_t others = !sure && c != chunk ? cost : 0xFFFFFFFFu;
    const int at_other = least(others);
    other = (uint32_t)__builtin_amdgcn_readlane((int)others, at_other) == 0xFFFFFFFFu ? 0u : (uint32_t)__builtin_amdgcn_readlane((int)c, at_other);
  }
  // The chunks have `items` items.  False: they are taken.  True: `chunk` is another length, to be counted: that of another
  // number of items per workgroup, then longer ones while they can still be better, then the best of all if it was not the last.
  // (Made longer only, 744 lists of 61 entries on average ended at 256: 16.6 us, now 15.0; 1088 of 82 at 320: 27.1 and 19.6, times
  // of lists that rows beyond decode_whole's bound hold.)
  __device__ __forceinline__ bool again(uint32_t items) {
    if (state == 5 || (state == 0 && items <= rounds * W)) return false;
    const uint32_t cost = (items + W - 1u) / W * (chunk + DEC_ITEM_ROWS) + DEC_CUT_ROWS;
    if (cost < best || (cost == best && chunk > best_chunk)) { best = cost; best_chunk = chunk; }
    if (++state == 1) {
      if (other) { chunk = other; return true; }
      ++state;
    }
    if (state < 5) {
      longer = decode_longer(longer);
      if (rounds * (longer + DEC_ITEM_ROWS) + DEC_CUT_ROWS < best) { chunk = longer; return true; }
    }
    state = 5;
    if (chunk == best_chunk) return false;
    chunk = best_chunk;
    return true;
  }
};

// What bounds it: few and short lists the chain length -> list entry -> page table -> K/V row -> merge, so every wave
// makes the item map and looks its rows up by itself and the only barrier of an item is the merge's (1 x 4096 tokens 5.9 ->
// 4.7 us, 4 x 16384 8.6 -> 7.3; with the map, the rows and the running maxima passed around the workgroup through LDS
// it took four and one more per 64 rows).  Long ones HBM, as long as loads keep going out: with a step's rows waited for,
// used and only then followed by the next step's, dense attention over 8 x 32768 tokens read 5.6 TB/s, now 6.2 (192 -> 173
// us), and 32 x 32768 gathered rows take 30.5 instead of 31.8.  Three workgroups per CU with four query heads per KV head:
// the registers of four (128) do not hold the addresses of the rows asked for ahead.
//
// WHOLE: every list is one item, of a workgroup of NW waves, and its result final: no item map, no partial results, no combine
// launch.  For lists that cannot be long (decode_whole).
template <int G, int NW = 4, bool WHOLE = false>
__global__ __launch_bounds__(64 * NW, NW == 8 || G == 8 ? 2 : (G == 4 ? 3 : 4)) void sparse_decode_kernel(DecodeArgs a) {
  constexpr int R = (G + 3) / 4;                 // score values a lane ends up owning per step
  constexpr int NT = 64 * NW, STEP = 16 * NW;    // entries of a step of the waves
  static_assert(WHOLE || (NW == 4 && STEP == (int)DEC_UNIT), "the item map is made by four waves");
  extern __shared__ int32_t prefix[];            // [NG + 1]
  __shared__ uint32_t wsum[16];
  __shared__ uint2 sum_s[4];
  __shared__ float2 macc[NW][G][64];             // the waves' accumulators ...
  __shared__ float2 ml_s[NW][G];                 // ... and their (maximum, denominator)
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), seg = tid & 15, row = lane >> 4;
  const bool dense = a.union_idx == nullptr;
  const bool b3 = seg & 8, b2 = seg & 4, b1 = seg & 2, b0 = seg & 1;
  const int my_t = seg >> 2;
  TW_STAMP(0);
  const int most = dense ? a.max_pages * TW_PAGE : a.union_stride;      // longest list
  auto length = [&](int gi) -> uint32_t {
    const int v = (dense ? a.seq_lens : a.union_count)[dense ? gi / a.LH : gi];
    return (uint32_t)(v < 0 ? 0 : (v > most ? most : v));
  };

  // ---- chunk length, item map (exclusive prefix of the lists' chunk counts) and this workgroup's first item
  const uint32_t W = gridDim.x;
  uint32_t chunk;
  int total_items, item = blockIdx.x, gi = 0, ck = 0, nchunks = 0;
  if constexpr (WHOLE) {
    chunk = (uint32_t)most;
    total_items = a.NG; nchunks = 1;
    gi = item;
  } else if (a.NG <= 64) {                        // block-uniform: lane l of every wave holds list l, no barrier
    const uint32_t c = lane < a.NG ? length(lane) : 0u;
    uint32_t rounds;
    chunk = decode_chunk((uint32_t)__builtin_amdgcn_readlane((int)tw_wave_scan_u32(c), 63), (uint32_t)a.NG, W, (uint32_t)a.chunk0, &rounds);
    uint32_t n = 0, incl = 0;
#pragma unroll 1
    for (int trial = 0; trial < 4; ++trial) {
      if (trial) chunk = decode_longer(chunk);
      n = (c + chunk - 1u) / chunk;
      incl = tw_wave_scan_u32(n);
      total_items = __builtin_amdgcn_readlane((int)incl, 63);
      if ((uint32_t)total_items <= rounds * W) break;
    }
    // the last lane that begins at or before the item (lanes of empty lists begin where the next one does)
    gi = __popcll(__ballot(incl - n <= (uint32_t)item)) - 1;
    ck = item - __builtin_amdgcn_readlane((int)(incl - n), gi);
    nchunks = __builtin_amdgcn_readlane((int)n, gi);
    if (wave == 0 && lane < a.NG) prefix[lane] = (int32_t)(incl - n);
    if (tid == 0) prefix[a.NG] = total_items;
  } else {                                        // thread t: the lists t * K ..
    // (more than two to a thread: read in whole lines, through LDS, K odd so that the lanes' words lie on different banks; read
    //  by their threads in every pass 6144 lists took 59.4 us, now 37.9; of lists in rows beyond decode_whole's bound)
    const int K1 = (a.NG + 255) >> 8, K = K1 > 2 ? K1 | 1 : K1, i0 = tid * K;
    uint32_t T = 0, longest = 0, c0 = 0, c1 = 0;
    if (K > 2) {
      for (int i = tid; i < a.NG; i += 256) {
        const uint32_t v = length(i);
        prefix[i] = (int32_t)v;
        T += v;
        longest = v > longest ? v : longest;
      }
    } else {
      c0 = i0 < a.NG ? length(i0) : 0u;
      c1 = K > 1 && i0 + 1 < a.NG ? length(i0 + 1) : 0u;
      T = c0 + c1;
      longest = c0 > c1 ? c0 : c1;
    }
    T = tw_wave_scan_u32(T);
    longest = tw_wave_max_u32(longest);
    if (lane == 63) sum_s[wave] = make_uint2(T, longest);
    __syncthreads();
    T = 0; longest = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint2 x = sum_s[w];
      T += x.x;
      longest = x.y > longest ? x.y : longest;
    }
    // One query head per KV head, 128 lists and more of 144 entries and more on average: no items of a single step.  A second
    // step's rows arrive behind the first's, and half as many workgroups share a CU and write pieces.  Attention with combine, us,
    // shortest chunk 64 / 128: 256 lists of 160 entries 11.8 / 10.9, 320 of 151 13.1 / 12.0, 320 of 210 14.0 / 13.3, 128 of 160
    // 9.5 / 8.8, 160 of 196 11.2 / 11.2; shorter or fewer lists leave the chip idle: 256 of 65 9.8 / 10.3, 224 of 129 10.2 / 10.4,
    // 96 of 299 10.4 / 10.8.
    const bool longer = G == 1 && a.kv_div == 1 && a.NG >= 128 && T >= 144u * (uint32_t)a.NG;
    DecodePlan plan(T, longest, (uint32_t)a.NG, W, longer ? max((uint32_t)a.chunk0, 2u * DEC_UNIT) : (uint32_t)a.chunk0);
    auto len_of = [&](int k) -> uint32_t { return K > 2 ? (i0 + k < a.NG ? (uint32_t)prefix[i0 + k] : 0u) : (k ? c1 : c0); };
    uint32_t n = 0, incl = 0, total;
#pragma unroll 1
    do {                                          // (block-uniform)
      n = 0;
      for (int k = 0; k < K; ++k) n += (len_of(k) + plan.chunk - 1u) / plan.chunk;
      incl = tw_block_scan_u32(n, wsum, &total);
    } while (plan.again(total));
    chunk = plan.chunk;
    n = incl - n;
    for (int k = 0; k < K; ++k) {
      const uint32_t v = len_of(k);
      if (i0 + k < a.NG) prefix[i0 + k] = (int32_t)n;
      n += (v + chunk - 1u) / chunk;
    }
    total_items = (int)total;
    if (tid == 0) prefix[a.NG] = total_items;
    __syncthreads();
  }
  if (!WHOLE && blockIdx.x == 0) {                // for the combine kernel
    __syncthreads();
    for (int i = tid; i <= a.NG; i += 256) a.ws_prefix[i] = prefix[i];
  }
  TW_STAMP(1);
  // list of an item: the last one with prefix <= item (empty lists begin where the next one does)
  auto find = [&]() {
    if (WHOLE) { gi = item; return; }
    int lo = 0, hi = a.NG;
    while (hi - lo > 1) { const int mid = (lo + hi) >> 1; if (prefix[mid] <= item) lo = mid; else hi = mid; }
    gi = lo; ck = item - prefix[lo]; nchunks = prefix[lo + 1] - prefix[lo];
  };
  if (item >= total_items) return;
  if (!WHOLE && a.NG > 64) find();

#pragma unroll 1
  for (;;) {
    const int b = gi / a.LH, l = gi % a.LH, g = l / a.kv_div;   // list l of sequence b, KV head g
    // Everything the row lookup reads that does not depend on another load goes out together: the sequence's length,
    // the list's length, this lane's list entry - any entry of the list's row may be read, those at or beyond the
    // count are ignored below - and q.  The page-table entries then depend on the list entries, the K/V rows on those:
    // three round trips to memory per item.
    // In a row of 16 lanes, lane seg looks up entry (seg % 4) * 4 * NW + wave * 4 + row of a step's 16 * NW.
    const int t0 = ck * (int)chunk;
    const int e0 = (seg & 3) * (STEP / 4) + wave * 4 + row;
    int nseq = a.seq_lens[b];                    // list entries at or beyond the sequence's end are ignored
    const int32_t* const cnt_p = dense ? a.seq_lens + b : a.union_count + gi;
    int cnt = *cnt_p;
    // (dense: the same loads from an address that is always valid, their values unused)
    const int32_t* const list = dense ? a.seq_lens + b : a.union_idx + (long long)gi * a.union_stride;
    const int list_end = dense ? 0 : a.union_stride - 1;
    auto entry = [&](int e) -> int { return list[t0 + e < list_end ? t0 + e : list_end]; };
    int raw0 = entry(e0), raw1 = entry(e0 + STEP), raw2 = entry(e0 + 2 * STEP);
    // q of the G heads, this lane's 8 dims, as loaded (bf16 pairs)
    uint4 q[G];
#pragma unroll
    for (int h = 0; h < G; ++h) q[h] = a.q[((long long)(b * a.Hq + l * G + h)) * 16 + seg];
    // (keeps the list-entry loads up here: the compiler would otherwise move them down to their first use, behind the
    //  wait for the two lengths)
    asm volatile("" : "+v"(raw0), "+v"(raw1), "+v"(raw2));
    if (nseq > a.max_pages * TW_PAGE) nseq = a.max_pages * TW_PAGE;
    if (dense) cnt = nseq;
    else if (cnt > a.union_stride) cnt = a.union_stride;
    nseq = __builtin_amdgcn_readfirstlane(nseq);
    const int len = __builtin_amdgcn_readfirstlane(cnt - t0 < (int)chunk ? cnt - t0 : (int)chunk);   // (scalar: what depends on it branches without lane masks)
    // entry e, read as r -> token (-1: does not count) -> the place of its page -> pool row.  (In three steps, so that
    // a load is not waited for before its value is needed.)
    auto token = [&](int r, int e) -> int {
      const int tk = dense ? t0 + e : r;
      return e < len && tk >= 0 && tk < nseq ? tk : -1;
    };
    auto page = [&](int tk) -> int { return a.page_table[(long long)b * a.max_pages + (tk < 0 ? 0 : tk >> 4)]; };
    auto pool_row = [&](int tk, int pp) -> int {
      return tk >= 0 && pp >= 0 && pp < a.pool_pages ? (pp * a.Hkv + g) * TW_PAGE + (tk & 15) : -1;
    };
    int tok = token(raw0, e0), pp = page(tok);
    const int tok1 = token(raw1, e0 + STEP), pp1 = page(tok1);
    int ids = pool_row(tok, pp);
    tok = tok1; pp = pp1;
    if (item == 0) TW_STAMP(2);
    float acc[G][8], M[R], lacc[R];
#pragma unroll
    for (int h = 0; h < G; ++h)
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[h][i] = 0.f;
#pragma unroll
    for (int r = 0; r < R; ++r) { M[r] = kNegBig; lacc[r] = 0.f; }

    // this wave's steps: those with at least one entry.  The next step's K rows are asked for as soon as this step's dot
    // products are done, its V rows behind this step's sums, so that a wave's loads keep going out while it computes -
    // in the registers of the rows just used.  (Unconditional loads, or a wait for one step's rows would take in the
    // next one's: entries that do not count all read the same 16 bytes and are masked.)
    const int steps = (len - wave * 4 + STEP - 1) >> (NW == 8 ? 7 : 6);
    if (steps > 0) {                              // (wave-uniform)
      const int own = __builtin_amdgcn_readfirstlane(ids), spare = own < 0 ? 0 : own;
      uint4 kr[4], vr[4];
      int rr[4];                                 // pool rows of the step whose K rows were asked for last, -1: none
      auto spread = [&]() {
        rr[0] = tw_row_bcast_i<0>(ids); rr[1] = tw_row_bcast_i<1>(ids); rr[2] = tw_row_bcast_i<2>(ids); rr[3] = tw_row_bcast_i<3>(ids);
      };
      auto ask = [&](uint4 (&x)[4], const uint4* pool) {
#pragma unroll
        for (int t = 0; t < 4; ++t) x[t] = tw_ld_stream(pool + (rr[t] < 0 ? (long long)spare * 16 : (long long)rr[t] * 16 + seg));
      };
      spread();
      ask(kr, a.k_pool);
      ask(vr, a.v_pool);
#ifdef TW_PHASE_TIMING
      if (item == 0) { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); TW_STAMP(3); }
#endif
#pragma unroll 1
      for (int st = 0; st < steps; ++st) {
        const bool valid = (my_t == 0 ? rr[0] : (my_t == 1 ? rr[1] : (my_t == 2 ? rr[2] : rr[3]))) >= 0;
        const bool void0 = rr[0] < 0, void1 = rr[1] < 0, void2 = rr[2] < 0, void3 = rr[3] < 0;
        // the pool rows of step st + 1, whose page-table entries were asked for a step ago; those of step st + 2 and the
        // list entries of step st + 3 are asked for
        ids = pool_row(tok, pp);
        tok = token(raw2, (st + 2) * STEP + e0);
        pp = page(tok);
        raw2 = entry((st + 3) * STEP + e0);
        // ---- partial dot products of this lane's 8 dims: val[t*4 + h%4][h/4]
        float val[16][R];
#pragma unroll
        for (int c = 0; c < 16; ++c)
#pragma unroll
          for (int r = 0; r < R; ++r) val[c][r] = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t) {
#pragma unroll
          for (int h = 0; h < G; ++h)              // bf16 pair dot products, fp32 accumulation
            val[t * 4 + (h & 3)][h >> 2] =
                tw_dot2_bf16(q[h].w, kr[t].w, tw_dot2_bf16(q[h].z, kr[t].z, tw_dot2_bf16(q[h].y, kr[t].y, tw_dot2_bf16(q[h].x, kr[t].x, 0.f))));
        }
        spread();
        __builtin_amdgcn_sched_barrier(0);
        ask(kr, a.k_pool);
        __builtin_amdgcn_sched_barrier(0);
        // ---- transposing reduction over the 16 lanes of the row: each step a lane keeps the half
        //      of the values selected by one bit of its lane id and adds the partner's copy of it;
        //      lane c ends with the full sum of value c
        float s_mine[R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float a8[8], a4[4], a2[2];
#pragma unroll
          for (int j = 0; j < 8; ++j) {
            const float keep = b3 ? val[j + 8][r] : val[j][r], send = b3 ? val[j][r] : val[j + 8][r];
            a8[j] = keep + tw_dpp_f<TW_DPP_MIRROR>(send);
          }
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float keep = b2 ? a8[j + 4] : a8[j], send = b2 ? a8[j] : a8[j + 4];
            a4[j] = keep + tw_dpp_f<TW_DPP_HALF_MIRROR>(send);
          }
#pragma unroll
          for (int j = 0; j < 2; ++j) {
            const float keep = b1 ? a4[j + 2] : a4[j], send = b1 ? a4[j] : a4[j + 2];
            a2[j] = keep + tw_dpp_f<TW_DPP_XOR2>(send);
          }
          const float keep = b0 ? a2[1] : a2[0], send = b0 ? a2[0] : a2[1];
          s_mine[r] = (keep + tw_dpp_f<TW_DPP_XOR1>(send)) * kLog2eRsqrtD;   // base-2 logit
        }
        // ---- running maximum per head of this lane, over the wave's 16 entries
        float sc[R], p_mine[R];
        bool moved = false;
#pragma unroll
        for (int r = 0; r < R; ++r) {
          float mx = valid ? s_mine[r] : -__builtin_inff();
          mx = fmaxf(mx, tw_dpp_f<TW_DPP_ROR4>(mx));
          mx = fmaxf(mx, tw_dpp_f<TW_DPP_ROR8>(mx));
          const float mn = fmaxf(M[r], tw_rows_max(mx));
          sc[r] = tw_exp2(M[r] - mn);
          moved |= M[r] != mn;
          M[r] = mn;
          p_mine[r] = valid ? tw_exp2(s_mine[r] - mn) : 0.f;
          lacc[r] = __builtin_fmaf(lacc[r], sc[r], p_mine[r]);
        }
        if (st > 0 && __any(moved)) {              // (wave-uniform)
#pragma unroll
          for (int h = 0; h < G; ++h) {
            const float f = (h & 3) == 0 ? tw_row_bcast<0>(sc[h >> 2]) : (h & 3) == 1 ? tw_row_bcast<1>(sc[h >> 2])
                          : (h & 3) == 2 ? tw_row_bcast<2>(sc[h >> 2]) : tw_row_bcast<3>(sc[h >> 2]);
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[h][i] *= f;
          }
        }
        // ---- every lane needs the 4 x G weights of its row: broadcast them lane by lane
        float pb[16][R];
#pragma unroll
        for (int r = 0; r < R; ++r) {
          pb[0][r] = tw_row_bcast<0>(p_mine[r]);   pb[1][r] = tw_row_bcast<1>(p_mine[r]);
          pb[2][r] = tw_row_bcast<2>(p_mine[r]);   pb[3][r] = tw_row_bcast<3>(p_mine[r]);
          pb[4][r] = tw_row_bcast<4>(p_mine[r]);   pb[5][r] = tw_row_bcast<5>(p_mine[r]);
          pb[6][r] = tw_row_bcast<6>(p_mine[r]);   pb[7][r] = tw_row_bcast<7>(p_mine[r]);
          pb[8][r] = tw_row_bcast<8>(p_mine[r]);   pb[9][r] = tw_row_bcast<9>(p_mine[r]);
          pb[10][r] = tw_row_bcast<10>(p_mine[r]); pb[11][r] = tw_row_bcast<11>(p_mine[r]);
          pb[12][r] = tw_row_bcast<12>(p_mine[r]); pb[13][r] = tw_row_bcast<13>(p_mine[r]);
          pb[14][r] = tw_row_bcast<14>(p_mine[r]); pb[15][r] = tw_row_bcast<15>(p_mine[r]);
        }
        if (__any(void0 | void1 | void2 | void3)) {              // (wave-uniform; the weights are 0, the row need not be finite)
          if (void0) vr[0] = make_uint4(0, 0, 0, 0);
          if (void1) vr[1] = make_uint4(0, 0, 0, 0);
          if (void2) vr[2] = make_uint4(0, 0, 0, 0);
          if (void3) vr[3] = make_uint4(0, 0, 0, 0);
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          float vf[8];
          tw_unpack8(vr[t], vf);
#pragma unroll
          for (int h = 0; h < G; ++h)
#pragma unroll
            for (int i = 0; i < 8; ++i) acc[h][i] = __builtin_fmaf(pb[t * 4 + (h & 3)][h >> 2], vf[i], acc[h][i]);
        }
        __builtin_amdgcn_sched_barrier(0);
        ask(vr, a.v_pool);
      }
    }

    if (item == 0) TW_STAMP(4);
    // ---- sum over the wave's four rows, transposing: a lane ends with the two dims d = 2 * (seg * 4 + row), d + 1
#pragma unroll
    for (int h = 0; h < G; ++h) {
#pragma unroll
      for (int i = 0; i < 4; ++i) { tw_swap32(acc[h][i], acc[h][i + 4]); acc[h][i] += acc[h][i + 4]; }
#pragma unroll
      for (int i = 0; i < 2; ++i) { tw_swap16(acc[h][i], acc[h][i + 2]); acc[h][i] += acc[h][i + 2]; }
      macc[wave][h][seg * 4 + row] = make_float2(acc[h][0], acc[h][1]);
    }
#pragma unroll
    for (int r = 0; r < R; ++r) {
      float lr = lacc[r];
      lr += tw_dpp_f<TW_DPP_ROR4>(lr);
      lr += tw_dpp_f<TW_DPP_ROR8>(lr);
      lr = tw_rows_sum(lr);
      if (lane < 4 && r * 4 + lane < G) ml_s[wave][r * 4 + lane] = make_float2(M[r], lr);
    }
    __syncthreads();
    // ---- the waves: thread -> 2 adjacent output dims of one head
#pragma unroll
    for (int c2 = tid; c2 < G * 64; c2 += NT) {
      const int h = c2 >> 6, d2 = c2 & 63;
      float2 ml[NW];
#pragma unroll
      for (int w = 0; w < NW; ++w) ml[w] = ml_s[w][h];
      float mx = fmaxf(fmaxf(ml[0].x, ml[1].x), fmaxf(ml[2].x, ml[3].x));
#pragma unroll
      for (int w = 4; w < NW; ++w) mx = fmaxf(mx, ml[w].x);
      float ox = 0.f, oy = 0.f, L = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float f = tw_exp2(ml[w].x - mx);
        const float2 v = macc[w][h][d2];
        ox = __builtin_fmaf(v.x, f, ox); oy = __builtin_fmaf(v.y, f, oy);
        L = __builtin_fmaf(ml[w].y, f, L);
      }
      if (WHOLE || nchunks == 1) {              // the item is the whole list: final result
        const int qh = b * a.Hq + l * G + h;
        const float inv = L > 0.f ? 1.0f / L : 0.f;
        ((uint32_t*)a.out)[(long long)qh * 64 + d2] = tw_f32_to_bf16(ox * inv) | (tw_f32_to_bf16(oy * inv) << 16);
        if (a.lse && d2 == 0) a.lse[qh] = L > 0.f ? (mx + __log2f(L)) * kLn2 : -__builtin_inff();
      } else {
        const long long at = (long long)item * G + h;
        a.ws_acc[at * 64 + d2] = make_float2(ox, oy);
        if (d2 == 0) a.ws_ml[at] = make_float2(mx, L);
      }
    }
    if (item == 0) TW_STAMP(5);
    item += (int)gridDim.x;
    if (item >= total_items) break;
    __syncthreads();                            // macc / ml_s are reused
    find();
  }
  if (blockIdx.x == 0) TW_STAMP(6);
}

struct CombineArgs {
  const int32_t* ws_prefix;
  const float2* ws_ml;
  const float* ws_acc;        // [items][G][128]
  uint16_t* out;              // bf16 [b][Hq][128]
  float* lse;
  int Hq, Hkv, G;
};

// One 256-thread block per (sequence, query head): 8 item lanes x 32 lanes of
// 4 output dims.  Each item lane folds every 8th partial with a running
// maximum; the 8 lanes are then merged through LDS.
__global__ __launch_bounds__(256) void combine_kernel(CombineArgs a) {
  const int b = blockIdx.y, h = blockIdx.x, tid = threadIdx.x, il = tid >> 5, dl = tid & 31;
  const int g = h / a.G, hh = h % a.G, gi = b * a.Hkv + g, qh = b * a.Hq + h;
  const int i0 = a.ws_prefix[gi], i1 = a.ws_prefix[gi + 1];
  if (i1 - i0 == 1) return;                     // written by the decode kernel itself
  uint2* out2 = (uint2*)(a.out + (long long)qh * 128);
  if (i1 == i0) {                               // empty list
    if (il == 0) out2[dl] = make_uint2(0u, 0u);
    if (a.lse && tid == 0) a.lse[qh] = -__builtin_inff();
    return;
  }
  const float4* acc4 = (const float4*)a.ws_acc;
  float m = kNegBig, l = 0.f;
  float4 o = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
  for (int i = i0 + il; i < i1; i += 8) {
    const float2 ml = a.ws_ml[(long long)i * a.G + hh];
    const float4 v = acc4[((long long)i * a.G + hh) * 32 + dl];
    const float mn = fmaxf(m, ml.x);
    const float so = tw_exp2(m - mn), sn = tw_exp2(ml.x - mn);
    l = __builtin_fmaf(l, so, ml.y * sn);
    o.x = __builtin_fmaf(o.x, so, v.x * sn); o.y = __builtin_fmaf(o.y, so, v.y * sn);
    o.z = __builtin_fmaf(o.z, so, v.z * sn); o.w = __builtin_fmaf(o.w, so, v.w * sn);
    m = mn;
  }
  __shared__ float4 so4[8][32];
  __shared__ float2 sml[8];
  so4[il][dl] = o;
  if (dl == 0) sml[il] = make_float2(m, l);
  __syncthreads();
  if (il == 0) {
    float M = sml[0].x;
#pragma unroll
    for (int j = 1; j < 8; ++j) M = fmaxf(M, sml[j].x);
    float L = 0.f;
    float4 r = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float sc = tw_exp2(sml[j].x - M);
      const float4 v = so4[j][dl];
      L = __builtin_fmaf(sml[j].y, sc, L);
      r.x = __builtin_fmaf(v.x, sc, r.x); r.y = __builtin_fmaf(v.y, sc, r.y);
      r.z = __builtin_fmaf(v.z, sc, r.z); r.w = __builtin_fmaf(v.w, sc, r.w);
    }
    const float inv = L > 0.f ? 1.0f / L : 0.f;
    out2[dl] = make_uint2(tw_f32_to_bf16(r.x * inv) | (tw_f32_to_bf16(r.y * inv) << 16),
                          tw_f32_to_bf16(r.z * inv) | (tw_f32_to_bf16(r.w * inv) << 16));
    if (a.lse && dl == 0) a.lse[qh] = L > 0.f ? (M + __log2f(L)) * kLn2 : -__builtin_inff();
  }
}

// The grid is persistent (a workgroup strides over the items), so it must not exceed what is
// resident at once: workgroups that wait for a slot would start their share only after an
// earlier one has finished all of its own.
template <int G>
int decode_blocks_per_cu(size_t lds) {
  // read-only property of the kernel, cached for the LDS size last asked for (racing threads compute the same value)
  static std::atomic<unsigned long long> cache{0};               // (lds << 8) | occupancy
  const unsigned long long c = cache.load(std::memory_order_relaxed);
  if ((c & 0xFF) != 0 && (c >> 8) == lds) return (int)(c & 0xFF);
  int n = 0;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&n, sparse_decode_kernel<G>, 256, lds) != hipSuccess || n < 1) n = 1;
  n = n > 6 ? 6 : n;
  cache.store(((unsigned long long)lds << 8) | (unsigned)n, std::memory_order_relaxed);
  return n;
}

template <int G>
void launch_decode(const DecodeArgs& a, long long max_items, size_t lds, hipStream_t s) {
  long long grid = (long long)tw_num_cus() * decode_blocks_per_cu<G>(lds);
  if (grid > max_items) grid = max_items;
  if (grid < 1) grid = 1;
  TW_LAUNCH((sparse_decode_kernel<G>), dim3((unsigned)grid), dim3(256), lds, s, a);
}

// Lists that cannot be long take a workgroup each and need no combine launch, which costs a step 2.4 us, nor the item map (1.2 us of the
// kernel's chain): eight waves up to a list per CU, four beyond, where three workgroups share a CU.  How long a list is only the
// device knows; a workgroup takes 1.1 us for every 128 entries, so the line lies where one list as long as its row among many a
// sixteenth of it, which the cut form shares out, loses nothing: at 512 entries, 256 with eight query heads to a row, and where there
// are lists for half the CUs, so that cut ones would run no wider either, at 768 and 512.  Steps over caches larger than the last-level
// one, us, cut / whole, (lists, bound), such lists:
//   1 head to a row    (32, 512) 23.9 / 24.0  (32, 640) 24.9 / 25.7  (128, 768) 27.4 / 27.6  (512, 768) 32.2 / 31.5
//   2                  (64, 512) 24.0 / 23.7  (64, 640) 24.1 / 24.8  (136, 768) 26.2 / 25.8  (512, 768) 31.8 / 30.4
//   4                  (64, 512) 24.2 / 24.1  (64, 640) 24.3 / 24.6  (136, 768) 27.1 / 27.4  (512, 768) 40.8 / 38.7
//   8                  (64, 256) 26.2 / 24.7  (64, 384) 26.4 / 26.8  (136, 512) 30.9 / 30.5  (512, 512) 57.9 / 51.3
// and beyond the lines, caches as the steps before left them: 4 heads (264, 1024) 31.4 / 32.6, (264, 1280) 32.5 / 35.4, 8 heads
// (136, 640) 29.9 / 31.0, (136, 1280) 31.3 / 36.8, 1 head (256, 1280) 31.8 / 34.3.  Lists of log-uniform or equal lengths gain at and
// below the lines: 4 heads (264, 768) 34.1 / 30.4, 8 heads (264, 512) 43.7 / 38.0, 1 head (256, 448) 29.1 / 24.3, 43 x 1668 multi-head
// (1376, 208) 63.8 / 56.6.
bool decode_whole(int NG, int G, int stride) {
  const bool many = 2 * NG >= tw_num_cus();
  return stride <= (G == 8 ? (many ? 512 : 256) : many ? 768 : 512);
}
template <int G>
void launch_whole(const DecodeArgs& a, hipStream_t s) {
  if (a.NG <= tw_num_cus()) TW_LAUNCH((sparse_decode_kernel<G, 8, true>), dim3(a.NG), dim3(512), 0, s, a);
  else TW_LAUNCH((sparse_decode_kernel<G, 4, true>), dim3(a.NG), dim3(256), 0, s, a);
}

}  // namespace

#ifdef TW_PHASE_TIMING
extern "C" int twilight_debug_stamps_decode(unsigned long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(tw_dbg_stamps), sizeof(unsigned long long) * 64) == hipSuccess ? 0 : -1;
}
#endif

// The shortest chunk that decode_chunk may choose: a step of the four waves for sparse lists (many small items keep
// all CUs busy on short, latency-bound gathers), longer for the dense sweep.
int tw_decode_chunk(bool dense) {
#ifdef TW_TUNING                                 // tuning builds only: the shipped library reads no environment
  static const int c0 = getenv("TW_DECODE_C0") ? atoi(getenv("TW_DECODE_C0")) : 0;
  if (!dense && (c0 == 64 || c0 == 128 || c0 == 256 || c0 == 512)) return c0;
#endif
  return dense ? 256 : 64;
}

long long tw_decode_max_items(const TwDims& d, bool dense, int union_stride) {
  const int chunk = tw_decode_chunk(dense);
  const long long max_len = dense ? (long long)d.max_pages * TW_PAGE : union_stride;
  return (long long)d.batch * d.Hkv * ((max_len + chunk - 1) / chunk);
}

static int decode_impl(const twilight_kv_t* kv, const void* q, const int32_t* count, const int32_t* idx, int32_t stride,
                       void* out, float* lse, void* ws, size_t ws_bytes, void* stream, bool per_head) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !out || !kv->k_pool || !kv->v_pool) return TW_EINVAL;
  const bool dense = idx == nullptr;
  if (per_head && dense) return TW_EINVAL;
  if (!dense && (!count || stride <= 0)) return TW_EINVAL;
  // one list per KV head shared by its G query heads, or one list per query head
  const int LH = per_head ? d.Hq : d.Hkv, Gk = per_head ? 1 : d.G;
  const int NG = d.batch * LH;
  if (NG > 12000) return TW_EINVAL;             // item map must fit in LDS
  if (!ws || ws_bytes < twilight_workspace_bytes(per_head ? TW_WS_DECODE_PER_HEAD : TW_WS_DECODE, kv, 0, dense ? 0 : stride))
    return TW_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;

  const long long max_items = tw_decode_max_items(d, dense, stride) / d.Hkv * LH;
  const size_t head_bytes = (((size_t)(NG + 1) * 4) + 255) & ~(size_t)255;
  const size_t ml_bytes = (((size_t)max_items * Gk * 8) + 255) & ~(size_t)255;
  DecodeArgs a;
  a.q = (const uint4*)q; a.k_pool = (const uint4*)kv->k_pool; a.v_pool = (const uint4*)kv->v_pool;
  a.page_table = kv->page_table; a.seq_lens = kv->seq_lens;
  a.union_count = dense ? nullptr : count; a.union_idx = idx;
  a.out = (uint4*)out; a.lse = lse;
  a.ws_prefix = (int32_t*)ws;
  a.ws_ml = (float2*)((char*)ws + head_bytes);
  a.ws_acc = (float2*)((char*)ws + head_bytes + ml_bytes);
  a.Hq = d.Hq; a.Hkv = d.Hkv; a.max_pages = d.max_pages; a.union_stride = stride;
  a.LH = LH; a.kv_div = per_head ? d.G : 1;
  a.NG = NG; a.chunk0 = tw_decode_chunk(dense); a.pool_pages = d.pool_pages;
  const size_t lds = (size_t)(NG + 1) * 4;
  tw_prof_before(TW_K_DECODE, s);
  if (!dense && decode_whole(NG, Gk, stride)) {
    switch (Gk) {
      case 1: launch_whole<1>(a, s); break;
      case 2: launch_whole<2>(a, s); break;
      case 4: launch_whole<4>(a, s); break;
      default: launch_whole<8>(a, s); break;
    }
    return tw_prof_after(s);
  }
  switch (Gk) {
    case 1: launch_decode<1>(a, max_items, lds, s); break;
    case 2: launch_decode<2>(a, max_items, lds, s); break;
    case 4: launch_decode<4>(a, max_items, lds, s); break;
    default: launch_decode<8>(a, max_items, lds, s); break;
  }
  if (int e = tw_prof_after(s)) return e;

  CombineArgs c;
  c.ws_prefix = a.ws_prefix; c.ws_ml = a.ws_ml; c.ws_acc = (const float*)a.ws_acc;
  c.out = (uint16_t*)out; c.lse = lse; c.Hq = d.Hq; c.Hkv = LH; c.G = Gk;
  tw_prof_before(TW_K_COMBINE, s);
  TW_LAUNCH(combine_kernel, dim3(d.Hq, d.batch), dim3(256), 0, s, c);
  return tw_prof_after(s);
}

// Launch shape of the decode kernel for this cache shape (host only): workgroups of the persistent grid (before
// it is cut to the number of work items), the shortest chunk, and how many numbers of items per workgroup
// decode_chunk weighs.  For benchmarks that report the balance of the work list, where lists are cut (twilight_decode_whole).
static int plan_dims(const twilight_kv_t* kv, int which, TwDims* d, int* LH, int* Gk) {
  if (!kv) return TW_EINVAL;
  twilight_kv_t tmp = *kv;                       // the pointers are not needed here: check the shape fields only
  int dummy = 0;
  tmp.page_table = &dummy; tmp.seq_lens = &dummy;
  if (int e = tw_check_kv(&tmp, d)) return e;
  if (which != TW_WS_DECODE && which != TW_WS_DECODE_PER_HEAD) return TW_EINVAL;
  *LH = which == TW_WS_DECODE_PER_HEAD ? d->Hq : d->Hkv;
  *Gk = which == TW_WS_DECODE_PER_HEAD ? 1 : d->G;
  return TW_OK;
}

extern "C" int twilight_decode_plan(const twilight_kv_t* kv, int which, int32_t dense, int32_t* grid, int32_t* chunk0,
                                    int32_t* items_per_wg) {
  TwDims d;
  int LH, Gk;
  if (!grid || !chunk0 || !items_per_wg) return TW_EINVAL;
  if (int e = plan_dims(kv, which, &d, &LH, &Gk)) return e;
  const size_t lds = (size_t)(d.batch * LH + 1) * 4;
  int occ = 1;
  switch (Gk) {
    case 1: occ = decode_blocks_per_cu<1>(lds); break;
    case 2: occ = decode_blocks_per_cu<2>(lds); break;
    case 4: occ = decode_blocks_per_cu<4>(lds); break;
    default: occ = decode_blocks_per_cu<8>(lds); break;
  }
  *grid = tw_num_cus() * occ;
  *chunk0 = tw_decode_chunk(dense != 0);
  *items_per_wg = (int32_t)DEC_MAX_ROUNDS;
  return TW_OK;
}

extern "C" int twilight_decode_whole(const twilight_kv_t* kv, int which, int32_t union_stride) {
  TwDims d;
  int LH, Gk;
  if (union_stride <= 0) return TW_EINVAL;
  if (int e = plan_dims(kv, which, &d, &LH, &Gk)) return e;
  return decode_whole(d.batch * LH, Gk, union_stride) ? 1 : 0;
}

extern "C" int twilight_sparse_decode(const twilight_kv_t* kv, const void* q, const int32_t* union_count,
                                      const int32_t* union_idx, int32_t union_stride, void* out, float* lse,
                                      void* ws, size_t ws_bytes, void* stream) {
  return decode_impl(kv, q, union_count, union_idx, union_stride, out, lse, ws, ws_bytes, stream, false);
}

extern "C" int twilight_sparse_decode_per_head(const twilight_kv_t* kv, const void* q, const int32_t* kept_count,
                                               const int32_t* kept_idx, int32_t kept_stride, void* out, float* lse,
                                               void* ws, size_t ws_bytes, void* stream) {
  return decode_impl(kv, q, kept_count, kept_idx, kept_stride, out, lse, ws, ws_bytes, stream, true);
}
