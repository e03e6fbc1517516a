// Selection of the Kp largest entries of one row of fp32 scores by a whole workgroup (Section 4.1: the page
// selector's top-k; also the channel-sparse token selector's).  Shared by the selection kernels and by the per-head
// pruner kernel that selects its pages itself.
//
// A row of up to E * NT entries lives in registers: thread t holds the keys of entries e * NT + t (coalesced loads; the
// order e, then wave, then lane is the entries' order, which is what the ordered listing needs).  The Kp-th largest key
// is located by bucketing the live key interval linearly (one pass when the scores are spread out), narrowing to the
// bucket that holds it, and an exact rank computation once at most SEL_CAP candidates remain.
//
// What bounds it is the chain of block barriers and LDS round trips, so every wave scans the histogram and ranks the
// candidates on its own (the same result in each) instead of waiting for one that does: 4 barriers per row, where keys
// staged in LDS, with the crossing bucket, the rank and the list offsets handed around through LDS, took 8.  Against that
// form, when it was left: selection inside the per-head kernel 5.0 -> 4.1 us (32 heads x 256 pages 5.0 -> 3.7), page_select 6.7 -> 5.5 us
// at 128 heads x 1024 pages, 10.8 -> 9.0 at 256 x 8192, 47 -> 26 at 256 x 32768 entries (measured apart from the
// figures below, which do not continue these).
// With 8 and more keys per thread, and for what 16 waves do alike, it is the vector instructions (256 rows x 32768 entries: 2584 per wave,
// 81 for each of a lane's keys, issuing in 70 % of a CU's busy cycles; 2159 and 68 % since): the first pass, whose keys are all inside
// the interval, adds without a test or a branch per key, and of the lane that the threshold falls to the waves look at one bucket per
// lane instead of walking its 8 to 32.  256 rows, an eighth taken, us: 32768 entries 31.8 -> 27.8, 8192 10.2 -> 9.4; the step of one
// sequence of 8192 pages 45.8 -> 43.3.
//
// Slots beyond the row's length are skipped by the whole workgroup, so that a row costs what its own length does: one by
// one up to 8 slots per thread, in groups of 4 beyond.  (512 rows x 9000 entries with 16 slots 15.5 us in groups of 4,
// 17.3 in groups of 8, 15.7 in groups of 2; 256 rows x 24000 with 32 slots 22.7 -> 20.1.  Full rows of 32768
// have a body without the groups' branches: page_select_reg_kernel.)
#pragma once
#include "tw_common.h"

constexpr int SEL_REG_PAGES = 8192;      // rows up to here may be split over two launches by length
constexpr int SEL_REG_TWO = 16384;       // rows up to here run two 1024-thread workgroups per CU (16 keys a thread in 64 registers)
constexpr int SEL_REG_MAX = 32768;       // longest row whose keys fit in a workgroup's registers
constexpr int SEL_CAP = 64;              // candidates of the exact finish: one per lane
constexpr int SEL_GROUP = 4;             // slots skipped together where a thread has more than 8
// Words of the histogram of SNB buckets: bucket r, from the top, in word r, with 16 or more to a scanning lane four words further for
// every lane before its own, so that the lanes' 16-byte reads begin on different banks; 64 words for slots beyond the row.
constexpr int tw_sel_words(int SNB) { return SNB + (SNB >= 1024 ? 4 * 64 : 0) + 64; }
constexpr uint32_t SEL_ALL_EQ = 0xFFFFFFFFu;   // every key equal to the threshold is taken

// entries of a sequence's row and how many of them the budget asks for (UNIT = tokens per entry: 16 or 1)
template <int UNIT>
__device__ __forceinline__ void tw_select_sizes(int n, int B, int max_pages, int max_sel, int* P_out, int* K_out) {
  int P = n > 0 ? (n + UNIT - 1) / UNIT : 0;
  if (P > max_pages) P = max_pages;
  long long kp = B > 0 ? ((long long)B + UNIT - 1) / UNIT : 0;
  if (kp > P) kp = P;
  if (kp > max_sel) kp = max_sel;
  *P_out = P;
  *K_out = (int)kp;
}

// Key of a long row's entry (more than 8 per thread): order-preserving, at least 1 for an entry of the row, 0 beyond its end.
// (Comparisons with the row's length at every use kept 32 lane masks alive and spilled the 32-entry form's registers.)
__device__ __forceinline__ uint32_t tw_select_key(float v, bool in) {
  const uint32_t k = tw_float_key(v);
  return in ? (k > 1u ? k : 1u) : 0u;
}

// Long rows' keys leave no registers for anything else per entry: what one phase derived from them (buckets, comparisons)
// is derived again by the next instead of being kept - which the compiler does, into scratch memory, if it sees the same
// keys in both.
template <int E>
__device__ __forceinline__ void tw_forget(uint32_t (&key)[E]) {
  if (E > 8) {
#pragma unroll
    for (int e = 0; e < E; ++e) asm volatile("" : "+v"(key[e]));
  }
}

// f(e) for this thread's slots e * NT + t that the row reaches, by a block-uniform test per slot, or per group of
// SEL_GROUP slots where a thread has more than 8.
// skipped(e) for the others.
template <int NT, int E, class F, class S>
__device__ __forceinline__ void tw_each_slot(int P, F f, S skipped) {
  constexpr int GRP = E > 8 ? SEL_GROUP : 1;
#pragma unroll
  for (int g = 0; g < E; g += GRP) {
    if (g * NT < P) {
#pragma unroll
      for (int e = g; e < g + GRP; ++e) f(e);
    } else {
#pragma unroll
      for (int e = g; e < g + GRP; ++e) skipped(e);
    }
  }
}
template <int NT, int E, class F>
__device__ __forceinline__ void tw_each_slot(int P, F f) { tw_each_slot<NT, E>(P, f, [](int) {}); }

// Exclusive prefix over `entries` (<= 64 * Q) per-wave counts in LDS, computed by every wave on its own: entry
// 64 * q + l ends up in excl[q] of lane l.
template <int Q>
__device__ __forceinline__ void tw_seg_prefix(const uint32_t* cnt, int entries, uint32_t (&excl)[Q], uint32_t* total) {
  const int lane = threadIdx.x & 63;
  uint32_t base = 0;
#pragma unroll
  for (int q = 0; q < Q; ++q) {
    const uint32_t v = q * 64 + lane < entries ? cnt[q * 64 + lane] : 0u;
    const uint32_t incl = tw_wave_scan_u32(v);
    excl[q] = base + incl - v;
    base += (uint32_t)__builtin_amdgcn_readlane((int)incl, 63);
  }
  *total = base;
}

// Threshold of the Kp (0 < Kp < P) largest of the row's keys, ties to the lower index: the entries with a key above
// *T_out and the first *need_eq_out of those equal to it (SEL_ALL_EQ: all).  key[e] of thread t is entry e * NT + t (tw_select_key when E > 8, else the
// float's key, of any value beyond the row's end).
// Called by all NT threads of the workgroup; hist (16-byte aligned) and cand are LDS of the caller.  SB: first phase-stamp slot (timing builds).
template <int NT, int E, int SNB, int SB>
__device__ __forceinline__ void tw_select_threshold(uint32_t (&key)[E], int P, uint32_t Kp, uint32_t* hist /* [tw_sel_words(SNB)] */,
                                                    unsigned long long* cand /* [SEL_CAP] */, uint32_t* T_out, uint32_t* need_eq_out) {
  constexpr int NW = NT / 64, BPL = SNB / 64;         // waves; histogram buckets per lane of a scanning wave
  constexpr int LB = BPL == 8 ? 3 : (BPL == 16 ? 4 : 5);
  static_assert(BPL == (1 << LB), "SNB is 512, 1024 or 2048");
  constexpr int PAD = BPL >= 16 ? 4 : 0, LANE = BPL + PAD, BEYOND = 64 * LANE;     // words per scanning lane; the first word for slots beyond the row
  auto word = [&](int r) -> int { return PAD ? r + (r >> LB) * PAD : r; };
  const int tid = threadIdx.x, lane = tid & 63, wave = E > 8 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const auto live = [&](int e) { return E > 8 || e * NT + tid < P; };   // (more than 8: the key says so)
  __shared__ uint32_t red_lo[NW], red_hi[NW];
  __shared__ uint32_t sh_n;
  TW_STAMP(SB);

  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  tw_each_slot<NT, E>(E > 8 ? P : E * NT, [&](int e) {     // (up to 8: the test per lane says it all)
    if (!live(e)) return;
    // (more than 8: the minimum is over key - 1 until all waves' are in - the 0 beyond the row's end wraps round and does
    //  not count, and neither does a wave that holds nothing else)
    const uint32_t k = E > 8 ? key[e] - 1u : key[e];
    lo = k < lo ? k : lo;
    hi = key[e] > hi ? key[e] : hi;
  });
  lo = ~tw_wave_max_u32(~lo);
  hi = tw_wave_max_u32(hi);
  if (lane == 0) { red_lo[wave] = lo; red_hi[wave] = hi; }
  if (tid == 0) sh_n = 0;
  if (tid < SEL_CAP) cand[tid] = 0;
  for (int i = tid; i < BEYOND; i += NT) hist[i] = 0;
  __syncthreads();
  uint32_t klo = ~tw_row_max_u32(~red_lo[lane & (NW - 1)]) + (E > 8 ? 1u : 0u), khi = tw_row_max_u32(red_hi[lane & (NW - 1)]);
  klo = (uint32_t)__builtin_amdgcn_readfirstlane((int)klo);
  khi = (uint32_t)__builtin_amdgcn_readfirstlane((int)khi);

  constexpr bool KEEP = E <= 8;
  int kept_bk[KEEP ? E : 1];
  uint32_t need = Kp, T = 0, need_eq = 0;
  tw_forget<E>(key);
  TW_STAMP(SB + 1);
#pragma unroll 1
  for (int pass = 0;; ++pass) {
    if (klo == khi) { T = klo; need_eq = need; break; }                    // everything left ties
    const float smn = tw_key_to_float(klo), smx = tw_key_to_float(khi);
    const float scale = (float)SNB / (smx - smn);
    // Buckets are linear in the score's value while that works: a finite scale over a normal, finite span, and only
    // for the first passes.  Otherwise (spans in the subnormal range, infinite scores, finite ones whose difference
    // is not, NaN, rows that keep falling into one bucket) they are linear in the order-preserving key, which splits any
    // span of at least SNB keys SNB ways and resolves a shorter one exactly, so every pass narrows the interval.
    // (An infinite span makes the scale 0 and a place the conversion of 0 * inf, which no bound holds; a scale up to 3e38 is that
    // of a span of at least SNB / 3e38, a normal number.)
    const bool by_key = !(scale > 0.f && scale <= 3.0e38f) || pass >= 3;
    const uint32_t span = khi - klo;
    const int kshift = span < (uint32_t)SNB ? 0 : 32 - __clz(span) - (LB + 6);
    // place from the top, 0 .. SNB - 1, of a key inside the interval
    auto bucket_of = [&](uint32_t k) -> int {
      if (by_key) return (int)((khi - k) >> kshift);
      const int r = (int)((smx - tw_key_to_float(k)) * scale);
      return r < SNB - 1 ? r : SNB - 1;
    };
    // is entry e of this thread in bucket bkt?  (rows of up to 8 entries per thread keep the bucket numbers)
    auto in_bucket = [&](int e, int bkt) -> bool {
      if (KEEP) return kept_bk[KEEP ? e : 0] == bkt;
      return live(e) && key[e] - klo <= span && bucket_of(key[e]) == bkt;
    };
    if (pass > 0) {
      for (int i = tid; i < BEYOND; i += NT) hist[i] = 0;
      __syncthreads();
    }
    if (pass == 0 && !by_key) {                   // (block-uniform)
      // every key of the row is inside: no branch around the add, so that the keys' chains overlap; slots beyond the row count
      // in words of their own
      tw_each_slot<NT, E>(P, [&](int e) {
        const int r = min((int)((smx - tw_key_to_float(key[e])) * scale), SNB - 1);
        const bool in = E > 8 ? key[e] != 0u : e * NT + tid < P;
        if (KEEP) kept_bk[KEEP ? e : 0] = in ? r : -1;
        atomicAdd(&hist[in ? word(r) : BEYOND + lane], 1u);
      }, [&](int e) { if (KEEP) kept_bk[KEEP ? e : 0] = -1; });
    } else {
      tw_each_slot<NT, E>(P, [&](int e) {
        const bool in = live(e) && key[e] - klo <= span;
        const int r = bucket_of(key[e]);
        if (KEEP) kept_bk[KEEP ? e : 0] = in ? r : -1;
        if (in) atomicAdd(&hist[word(r)], 1u);
      }, [&](int e) { if (KEEP) kept_bk[KEEP ? e : 0] = -1; });
    }
    __syncthreads();
    TW_STAMP(SB + 2);
    // lane l sums the buckets BPL * l .. up; then, of the lane that the threshold falls to, one bucket per lane
    uint32_t mine = 0;
#pragma unroll
    for (int j = 0; j < BPL; j += 4) {
      const uint4 x = *(const uint4*)(hist + LANE * lane + j);
      mine += x.x + x.y + x.z + x.w;
    }
    const uint32_t above = tw_wave_scan_u32(mine) - mine;
    const int src = __ffsll((long long)__ballot(above < need && above + mine >= need)) - 1;   // the interval holds the threshold
    need -= (uint32_t)__builtin_amdgcn_readlane((int)above, src);
    const uint32_t c = lane < BPL ? hist[LANE * src + lane] : 0u;
    const uint32_t upto = tw_wave_scan_u32(c);
    const int at = __ffsll((long long)__ballot(upto >= need)) - 1;
    const int bkt = BPL * src + at;
    const uint32_t pop = (uint32_t)__builtin_amdgcn_readlane((int)c, at);
    need -= (uint32_t)__builtin_amdgcn_readlane((int)upto, at) - pop;
    tw_forget<E>(key);
    if (pop <= (uint32_t)SEL_CAP) {
      // exact: the bucket's keys, with the lower index the larger of two equals, ranked by every wave on its own - one
      // candidate per lane; the one of rank need - 1 is the last one taken
      tw_each_slot<NT, E>(KEEP ? E * NT : P, [&](int e) {
        const int i = e * NT + tid;
        if (in_bucket(e, bkt)) {
          const uint32_t at = atomicAdd(&sh_n, 1u);
          if (at < (uint32_t)SEL_CAP) cand[at] = ((unsigned long long)key[e] << 32) | (uint32_t)~i;
        }
      });
      __syncthreads();
      TW_STAMP(SB + 3);
      const unsigned long long mineK = cand[lane];                         // 0 beyond pop: below every candidate
      uint32_t rank = 0;
#pragma unroll 1
      for (uint32_t j0 = 0; j0 < pop; j0 += 8) {
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) rank += cand[j0 + j] > mineK ? 1u : 0u;
      }
      const int last = __ffsll((long long)__ballot((uint32_t)lane < pop && rank == need - 1)) - 1;
      T = (uint32_t)__builtin_amdgcn_readlane((int)(mineK >> 32), last);
      // how many of the keys equal to T are taken: those ranked up to `last`
      const unsigned long long eq = __ballot((uint32_t)lane < pop && (uint32_t)(mineK >> 32) == T);
      const unsigned long long in = eq & __ballot(rank <= need - 1);
      need_eq = in == eq ? SEL_ALL_EQ : (uint32_t)__popcll(in);
      break;
    }
    // narrow to the bucket's keys
    uint32_t nlo = 0xFFFFFFFFu, nhi = 0u;
    tw_each_slot<NT, E>(KEEP ? E * NT : P, [&](int e) {
      if (in_bucket(e, bkt)) {
        nlo = key[e] < nlo ? key[e] : nlo;
        nhi = key[e] > nhi ? key[e] : nhi;
      }
    });
    nlo = ~tw_wave_max_u32(~nlo);
    nhi = tw_wave_max_u32(nhi);
    if (lane == 0) { red_lo[wave] = nlo; red_hi[wave] = nhi; }
    __syncthreads();
    klo = (uint32_t)__builtin_amdgcn_readfirstlane((int)~tw_row_max_u32(~red_lo[lane & (NW - 1)]));
    khi = (uint32_t)__builtin_amdgcn_readfirstlane((int)tw_row_max_u32(red_hi[lane & (NW - 1)]));
    if (pop == need) { T = klo; need_eq = SEL_ALL_EQ; break; }    // the whole bucket is taken
    __syncthreads();                              // red_* and hist are rewritten by the next pass
  }
  tw_forget<E>(key);
  TW_STAMP(SB + 4);
  *T_out = T;
  *need_eq_out = need_eq;
}

// Ordered listing behind tw_select_threshold: put(pos, e) is called for every selected entry e * NT + t of this thread
// with its place in the ascending list.  cnt: LDS of the caller, E * NT / 64 words.  Called by all NT threads; one barrier.
template <int NT, int E, class Put>
__device__ __forceinline__ void tw_select_list(uint32_t (&key)[E], int P, uint32_t T, uint32_t need_eq, uint32_t* cnt, Put put) {
  constexpr int NW = NT / 64, SEGS = E * NW, Q = (SEGS + 63) / 64;
  const int tid = threadIdx.x, lane = tid & 63, wave = E > 8 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const auto live = [&](int e) { return E > 8 || e * NT + tid < P; };
  uint32_t excl[Q], total;
  // Block-uniform, and so but for ties that are cut: one comparison and one ballot per entry (instructions bound this
  // phase once 16 waves share a CU's four vector units: 256 x 32768 entries 32.0 -> 29.7 us, 32 heads x 8192 2.9 -> 2.4).
  if (need_eq == SEL_ALL_EQ) {
    static_assert(E <= 64, "a lane per slot");
    uint32_t mine = 0;                            // lane e: how many of this wave's slots e are taken
    tw_each_slot<NT, E>(P, [&](int e) {
      const uint32_t c = (uint32_t)__popcll(__ballot(live(e) && key[e] >= T));
      mine = lane == e ? c : mine;
    });
    if (lane < E) cnt[lane * NW + wave] = mine;
    __syncthreads();
    tw_forget<E>(key);
    tw_seg_prefix<Q>(cnt, ((P + NT - 1) / NT) * NW, excl, &total);
    tw_each_slot<NT, E>(P, [&](int e) {
      const bool in = live(e) && key[e] >= T;
      const uint32_t below = tw_bits_below(__ballot(in));
      if (in) put((uint32_t)__builtin_amdgcn_readlane((int)excl[(e * NW) >> 6], ((e * NW) & 63) + wave) + below, e);
    });
    return;
  }
  tw_each_slot<NT, E>(P, [&](int e) {
    const uint32_t gt = (uint32_t)__popcll(__ballot(live(e) && key[e] > T)), eq = (uint32_t)__popcll(__ballot(live(e) && key[e] == T));
    if (lane == 0) cnt[e * NW + wave] = gt | (eq << 16);
  });
  __syncthreads();
  tw_forget<E>(key);
  tw_seg_prefix<Q>(cnt, ((P + NT - 1) / NT) * NW, excl, &total);
  tw_each_slot<NT, E>(P, [&](int e) {
    const bool gt = live(e) && key[e] > T, eq = live(e) && key[e] == T;
    const unsigned long long bg = __ballot(gt), be = __ballot(eq);
    const uint32_t off = (uint32_t)__builtin_amdgcn_readlane((int)excl[(e * NW) >> 6], ((e * NW) & 63) + wave);
    const uint32_t gt_before = (off & 0xFFFFu) + tw_bits_below(bg), eq_before = (off >> 16) + tw_bits_below(be);
    if (gt || (eq && eq_before < need_eq)) put(gt_before + (eq_before < need_eq ? eq_before : need_eq), e);
  });
}
