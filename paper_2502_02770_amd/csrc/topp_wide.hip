// Stage 2b/c for long candidate rows (paper: Algorithm 1, Definition 3.3,
// Appendix B.2): the threshold set of the register-resident kernel, spread
// over many workgroups per head.  Used when a head has more than 8192
// candidates (every token a candidate - no selector in front - or very large
// budgets) or the sequence is too long for the in-LDS bitmap.
//
//   row_sample    (topp_prune.hip) scores a sample of the row, which places the head's histogram grid; clears the
//                 per-head histogram, counters and sums
//   (scoring      also folds the row maximum into headmax with atomicMax and the scores into the mass histogram)
//   wide_init, wide_hist   clearing, and grid and histogram from the stored scores: behind the scoring kernels that do
//                 not make the histogram themselves
//   wide_decide   one wave per head: the bucket or two of the histogram that the threshold falls into
//   wide_emit     one pass over the scores: those above the buckets -> bitmap, those inside -> a short per-head list,
//                 and the exact fixed-point masses of the row and of the scores above
//   wide_resolve  finds the exact threshold among the listed scores inside one workgroup (narrowing
//                 in LDS, then exact on the scores' own bits), sets their bits
//   bitmap_list   bitmap(s) -> ascending index list (per-head kept list, and
//                 the union of a KV head's query heads)
//
// What bounds it is the traffic of the score rows: written once by the scoring kernel and read once here.  Masses are
// relative to the row's largest score, which is known only when all are scored, so a histogram of exact masses would
// take a pass over the rows of its own; masses relative to a histogram grid are enough to say where the
// threshold lies, and wide_resolve checks that with the exact sums: a row whose threshold is not among its listed
// scores - or with more than W_CAP of them - is searched again from its scores by wide_resolve.
// At 4 x 64 heads x 262144 tokens: 322 -> 281 us for the whole pruner (scoring 177 -> 185, emit 52 as before, and no
// histogram passes: 55 us and four launches of 4 us that found nothing left to do).
//
// The deciding sums are 64-bit fixed point over the same terms in any order, so the sets do not depend on scheduling
// (nor on where the histogram cut).
#include <stdlib.h>
#include "topp_common.h"

namespace {

constexpr int W_SLOTS = 32;                    // candidate slots per thread
constexpr int W_CAP = WIDE_LIST_CAP;           // undecided scores that the resolve kernel takes

struct WideArgs {
  const float* scores;
  const int32_t* sel_pages;   // or nullptr
  const int32_t* sel_count;
  const int32_t* seq_lens;
  const uint32_t* headmax;    // [bh][HM_SLOTS] (padded): max = key of the head's largest score, 0 = no valid score
  unsigned long long* ghist;  // [bh][WH_NB]
  WhGrid* hgrid;              // [bh]
  float4* range;              // [bh] {largest score, d_hi, d_lo, -}
  unsigned long long* sums;   // [bh][WS_SUMS]: mass of the row, mass above the undecided range
  uint2* ulist;               // [bh][W_CAP] {key, token}
  uint32_t* ucount;
  uint32_t* kdef;
  uint32_t* bitmaps;
  int32_t* kept_count;
  uint32_t* status;
  int Hq, max_pages, max_sel, cand_stride, words_stride;
  int keep_all;               // p >= 1
  float p;
};

__global__ __launch_bounds__(256) void wide_init_kernel(uint4* zero_base, size_t n16) {
  const size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n16) zero_base[i] = make_uint4(0, 0, 0, 0);
}

// the head's largest score: maximum over the words the scoring workgroups folded into
__device__ __forceinline__ uint32_t wide_headmax(const uint32_t* headmax, int bh, int lane) {
  const uint32_t v = lane < HM_SLOTS ? headmax[((long long)bh * HM_SLOTS + lane) * TW_CTR] : 0u;
  return tw_wave_max_u32(v);
}

__device__ __forceinline__ int wide_count(const WideArgs& a, int b, int bh) {
  const int n = a.seq_lens[b];
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  int count = P;
  if (a.sel_pages) { count = a.sel_count[bh]; if (count > a.max_sel) count = a.max_sel; if (count < 0) count = 0; }
  return count;
}

// A workgroup of NT threads covers NT * W_SLOTS consecutive candidate slots; thread t owns 8 groups
// of 4 slots, group v at chunk + v * 4 * NT + 4t, so that every load instruction of a wave reads
// 1 KiB contiguous.  Loaded unconditionally (clamped) and masked to -inf at and beyond N.
template <int NT>
__device__ __forceinline__ int wide_slot(int chunk0, int v, int tid) { return chunk0 + v * 4 * NT + tid * 4; }
template <int NT>
__device__ __forceinline__ void wide_load(const float* row, int chunk0, int tid, int N, int cand_stride, float* s) {
#pragma unroll
  for (int v = 0; v < W_SLOTS / 4; ++v) {
    const int c = wide_slot<NT>(chunk0, v, tid);
    const float4 x = *(const float4*)(row + (c < cand_stride ? c : cand_stride - 4));
    s[4 * v] = c < N ? x.x : -__builtin_inff();     // N is a multiple of 16: a group is inside or outside
    s[4 * v + 1] = c < N ? x.y : -__builtin_inff();
    s[4 * v + 2] = c < N ? x.z : -__builtin_inff();
    s[4 * v + 3] = c < N ? x.w : -__builtin_inff();
  }
}

// Grid and histogram from the stored scores.  Every workgroup of a head takes the same sample of its row - 1024 scores
// evenly spread - so all lay the same grid; the first one leaves it for the passes that follow.
template <int NT>
__global__ __launch_bounds__(NT) void wide_hist_kernel(WideArgs a) {
  constexpr int W_CHUNK = NT * W_SLOTS, NW = NT / 64, K = 1024 / NT;
  const int bh = blockIdx.y, b = bh / a.Hq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int N = wide_count(a, b, bh) * TW_PAGE;
  if ((long long)blockIdx.x * W_CHUNK >= N) return;
  const int chunk0 = blockIdx.x * W_CHUNK;
  const float* const row = a.scores + (long long)bh * a.cand_stride;
  float sv[K];
#pragma unroll
  for (int k = 0; k < K; ++k) sv[k] = row[(int)(((long long)(k * NT + tid) * N) >> 10)];
  const float mx = tw_key_to_float(wide_headmax(a.headmax, bh, lane));
  __shared__ unsigned long long hist[WH_NB];
  __shared__ float sum_s[NW][3];
  for (int i = tid; i < WH_NB; i += NT) hist[i] = 0;
  float s[W_SLOTS];
  wide_load<NT>(row, chunk0, tid, N, a.cand_stride, s);
  float w0 = 0.f, w1 = 0.f, w2 = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (sv[k] > -__builtin_inff() && mx < __builtin_inff()) {
      const float t = sv[k] - mx, w = __expf(t);
      w0 += w; w1 += w * t; w2 += w * t * t;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { w0 += __shfl_xor(w0, o, 64); w1 += __shfl_xor(w1, o, 64); w2 += __shfl_xor(w2, o, 64); }
  if (lane == 0) { sum_s[wave][0] = w0; sum_s[wave][1] = w1; sum_s[wave][2] = w2; }
  __syncthreads();
  w0 = w1 = w2 = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) { w0 += sum_s[w][0]; w1 += sum_s[w][1]; w2 += sum_s[w][2]; }
  WhGrid gr = wh_grid(w0, w1, w2);
  if (w0 > 0.f) gr.ref += mx;
  if (blockIdx.x == 0 && tid == 0) a.hgrid[bh] = gr;
  const float inv = 1.0f / gr.scale, off = -gr.ref * inv, lscale = gr.scale * 0x1.715476p+0f;
#pragma unroll
  for (int e = 0; e < W_SLOTS; ++e) {
    uint32_t w;
    const bool valid = s[e] > -__builtin_inff();
    const int bk = wh_bucket(__builtin_fmaf(valid ? s[e] : 0.f, inv, off), lscale, &w);
    if (valid) atomicAdd(&hist[bk], (unsigned long long)w);
  }
  __syncthreads();
  for (int i = tid; i < WH_NB; i += NT) {
    const unsigned long long c = hist[i];
    if (c) atomicAdd(&a.ghist[(long long)bh * WH_NB + i], c);
  }
}

// The scores among which the head's threshold lies, by its histogram of N scores: distances to the maximum d_hi <= d < d_lo.
__device__ __forceinline__ void wide_range(const unsigned long long* gh, WhGrid gr, float m, float p, int N, int lane, float* d_hi, float* d_lo) {
  constexpr int BPL = WH_NB / 64;
  static_assert(WH_NB % 64 == 0, "whole buckets per lane");
  float mb[BPL], mine = 0.f;
#pragma unroll
  for (int k = 0; k < BPL; ++k) {
    const int bk = BPL * lane + k;
    const float t = bk < WH_HALF ? wh_edge(WH_HALF - bk) : -wh_edge(bk - WH_HALF);             // upper edge
    mb[k] = (float)gh[bk] * __expf(fminf(gr.ref + t * gr.scale - m, 80.f));
    mine += mb[k];
  }
  float incl = mine;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const float y = __shfl_up(incl, o, 64);
    if (lane >= o) incl += y;
  }
  const float Z = __shfl(incl, 63, 64);
  *d_hi = 0.f; *d_lo = HP_REACH;                         // a histogram that says nothing: everything is undecided
  if (!(Z > 0.f) || !(Z < __builtin_inff()) || __shfl(mb[0], 0, 64) > 0.f) return;     // wave-uniform
  // The buckets in which the kept mass may reach p of the whole, summed from the top down below p = 1/2 and from the bottom
  // up above: there the mass left out has to fall to 1 - p of the whole, and the sums' roundings are relative to it.
  // Margin: roundings of the weights (2^-19 of a bucket's edge) and of these sums, with much to spare; what the exact
  // masses, whole multiples of 2^-40, drop of each score, or of one beyond their reach (here in units of 2^-19); what lies
  // beyond the last bucket's edge.  (5e-5 of the whole mass whatever p is is more than p = 0.99999 leaves out: every score
  // below the threshold was then undecided, and peaked rows, whose tail is most of their scores, overflowed their lists;
  // without the second term some lists miss the threshold.  Logits of deviation 4, 32 heads x 131072 at p = 0.99999 and
  // 0.999999: 107 -> 30 and 32 us of top-p, 256 x 262144 at p = 0.9999 and 0.99999: 285 -> 86 and 316 -> 90, 219 without
  // the second term.)
  const float left = 1.f - p;
  const float eps = fminf(5e-5f, 1e-3f * left) * Z + (float)N * 0x1p-20f + __shfl(mb[BPL - 1], 63, 64);
  int b0 = WH_NB, b1 = WH_NB;
  if (p < 0.5f) {
    const float t0 = p * Z - eps, t1 = p * Z + eps;
    float cum = incl - mine;
#pragma unroll
    for (int k = 0; k < BPL; ++k) {
      cum += mb[k];
      if (b0 == WH_NB && cum >= t0) b0 = BPL * lane + k;
      if (b1 == WH_NB && cum >= t1) b1 = BPL * lane + k;
    }
  } else {
    float below = mine;                                  // mass of this lane's buckets and of those below them
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const float y = __shfl_down(below, o, 64);
      if (lane + o < 64) below += y;
    }
    below = __shfl_down(below, 1, 64);
    if (lane == 63) below = 0.f;
    const float t0 = left * Z + eps, t1 = left * Z - eps;
#pragma unroll
    for (int k = BPL - 1; k >= 0; --k) {
      if (below <= t0) b0 = BPL * lane + k;
      if (below <= t1) b1 = BPL * lane + k;
      below += mb[k];
    }
  }
  const unsigned long long h0 = __ballot(b0 < WH_NB), h1 = __ballot(b1 < WH_NB);
  b0 = h0 ? __shfl(b0, __ffsll((long long)h0) - 1, 64) : WH_NB - 1;
  b1 = h1 ? __shfl(b1, __ffsll((long long)h1) - 1, 64) : WH_NB - 1;
  // In steps of 2^-10 logits: whole ranks (2^-22), so that scores of one rank, which may end as one tier, stay together.
  if (b0 > 0) {
    const float t = b0 < WH_HALF ? wh_edge(WH_HALF - b0) : -wh_edge(b0 - WH_HALF);             // upper edge of b0
    const float d = floorf((m - (gr.ref + t * gr.scale)) * 1024.f) * 0.0009765625f;
    *d_hi = fminf(fmaxf(d, 0.f), HP_REACH);
  }
  if (b1 < WH_NB - 1) {
    const float t = b1 < WH_HALF ? wh_edge(WH_HALF - 1 - b1) : -wh_edge(b1 + 1 - WH_HALF);     // lower edge of b1
    const float d = ceilf((m - (gr.ref + t * gr.scale)) * 1024.f) * 0.0009765625f;
    *d_lo = fminf(fmaxf(d, 0.f), HP_REACH);
  }
}

// (A launch of its own: in the prologue of every wide_emit workgroup this made that kernel 81 us instead of 52 + this one's 4.8.)
__global__ __launch_bounds__(64) void wide_decide_kernel(WideArgs a) {
  const int bh = blockIdx.x, lane = threadIdx.x;
  const int N = wide_count(a, bh / a.Hq, bh) * TW_PAGE;
  const float m = tw_key_to_float(wide_headmax(a.headmax, bh, lane));   // (no valid score: a NaN, nothing takes part)
  float d_hi = 0.f, d_lo = HP_REACH;
  wide_range(a.ghist + (long long)bh * WH_NB, a.hgrid[bh], m, a.p, N, lane, &d_hi, &d_lo);
  if (lane == 0) a.range[bh] = make_float4(m, d_hi, d_lo, 0.f);
}

// Two words that are the same in all lanes, to one lane.  (The wait is the one from a comparison's lane mask to its use by a vector instruction.)
__device__ __forceinline__ void wide_to_lane(int lane, unsigned long long x, uint32_t& lo, uint32_t& hi) {
  asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4" : "+v"(lo), "+v"(hi) : "s"((uint32_t)x), "s"((uint32_t)(x >> 32)), "n"(lane));
}

// A wave covers 64 * W_SLOTS consecutive slots, 64 at a time, so that a comparison's lane mask is two words of the bitmap.
// What bounds it is vector instructions, then the read of the rows.  Masses, floor(e * 2^40), are summed by one
// 64-bit fma each, rounded towards zero in an accumulator between 2^52 and 2^53, whose last place is 1: the integers' sum, exactly.
// (As two 20-bit parts, with the flags gathered per lane and joined across lanes, 30 instructions a score; 15 so.  4 x 64 heads x
// 262144, in a kernel trace of the pruner's steps, 55.6 -> 52.2 us, 268 MB at 5.1 TB/s; by events around the launch 51.9 -> 46.4,
// 4 x 32 heads 29.2 -> 24.9, 1 x 64 17.0 -> 14.8, 16 x 32 x 32768 17.3 -> 15.0.)
template <int NT>
__global__ __launch_bounds__(NT) void wide_emit_kernel(WideArgs a) {
  constexpr int W_CHUNK = NT * W_SLOTS, NW = NT / 64;
  const int bh = blockIdx.y, b = bh / a.Hq, tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int count = wide_count(a, b, bh);
  const int N = count * TW_PAGE;
  if ((long long)blockIdx.x * W_CHUNK >= N) return;
  const int w0 = blockIdx.x * W_CHUNK + wave * 64 * W_SLOTS;       // this wave's first slot
  const float* const row = a.scores + (long long)bh * a.cand_stride;
  float s[W_SLOTS];
  if (w0 + 64 * W_SLOTS <= N) {                   // (wave-uniform)
#pragma unroll
    for (int e = 0; e < W_SLOTS; ++e) s[e] = row[w0 + e * 64 + lane];
  } else {
#pragma unroll
    for (int e = 0; e < W_SLOTS; ++e) s[e] = row[w0 + e * 64 + lane < N ? w0 + e * 64 + lane : N - 1];
#pragma unroll
    for (int e = 0; e < W_SLOTS; ++e) s[e] = w0 + e * 64 + lane < N ? s[e] : -__builtin_inff();
  }
  const float4 rg = a.range[bh];
  const float m = rg.x, d_hi = rg.y, d_lo = rg.z;
  uint32_t klo = 0, khi = 0, ulo = 0, uhi = 0;    // lane e: the kept and the undecided of the slots w0 + 64 * e .. up
  uint32_t cnt = 0;                               // kept (wave-uniform)
  uint32_t any = 0;
  double Zd, Ad;
  asm volatile("s_setreg_imm32_b32 hwreg(HW_REG_MODE, 2, 2), 3" ::: "memory");    // 64-bit results towards zero, to the kernel's end
  {
    unsigned long long one = 0x4330000000000000ull;                               // 2^52
    asm volatile("" : "+v"(one));
    Zd = Ad = __builtin_bit_cast(double, one);
  }
  if (a.keep_all) {
#pragma unroll
    for (int e = 0; e < W_SLOTS; ++e) {
      const unsigned long long keep = __ballot(s[e] > -__builtin_inff());
      cnt += (uint32_t)__popcll(keep);
      wide_to_lane(e, keep, klo, khi);
    }
  } else {
#pragma unroll
    for (int e = 0; e < W_SLOTS; ++e) {
      const float d = __fsub_rn(m, s[e]);
      const float x = __expf(-(d < HP_REACH ? d : 100.f));         // beyond the reach: no mass
      const bool kept = d < d_hi;
      asm("v_fma_f64 %0, %1, %2, %0" : "+v"(Zd) : "v"((double)x), "s"(0x1p40));
      asm("v_fma_f64 %0, %1, %2, %0" : "+v"(Ad) : "v"((double)(kept ? x : 0.f)), "s"(0x1p40));
      const unsigned long long keep = __ballot(kept), und = __ballot(d < d_lo) & ~keep;
      cnt += (uint32_t)__popcll(keep);
      wide_to_lane(e, keep, klo, khi);
      if (und) { any = 1; wide_to_lane(e, und, ulo, uhi); }        // (wave-uniform)
    }
  }
  unsigned long long Z = __builtin_bit_cast(unsigned long long, Zd) & 0xFFFFFFFFFFFFFull, A = __builtin_bit_cast(unsigned long long, Ad) & 0xFFFFFFFFFFFFFull;
  // undecided scores go onto the head's list: one atomic per wave reserves room for all its lanes
  if (any) {                                      // wave-uniform
    const uint32_t mine = __popc(ulo) + __popc(uhi);
    const uint32_t incl = tw_wave_scan_u32(mine);
    uint32_t ubase = 0;
    if (lane == 63) ubase = atomicAdd(&a.ucount[(long long)bh * TW_CTR], incl);
    uint32_t at = __shfl(ubase, 63, 64) + incl - mine;
    // (few scores: their words are read again, so that none of the 32 has to stay in a register for this)
    for (unsigned long long x = ((unsigned long long)uhi << 32) | ulo; x; x &= x - 1, ++at) {
      const int slot = w0 + lane * 64 + __ffsll((long long)x) - 1;
      if (at < (uint32_t)W_CAP) {
        const int tok = a.sel_pages ? a.sel_pages[(long long)bh * a.max_sel + (slot >> 4)] * TW_PAGE + (slot & 15) : slot;
        a.ulist[(long long)bh * W_CAP + at] = make_uint2(tw_float_key(row[slot]), (uint32_t)tok);
      }
    }
  }
  uint32_t* bm = a.bitmaps + (long long)bh * a.words_stride;
  if (lane < W_SLOTS) {
    const int c = w0 + lane * 64;
    if (a.sel_pages) {                            // one 16-bit half word per selected page
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int pi = (c >> 4) + v;
        if (pi < count) {
          const int pg = a.sel_pages[(long long)bh * a.max_sel + pi];
          if (pg >= 0 && (pg >> 1) < a.words_stride)   // ids outside the row: no bits, no store
            ((unsigned short*)bm)[pg] = (unsigned short)((v < 2 ? klo : khi) >> (16 * (v & 1)));
        }
      }
    } else {                                      // slots are token positions
      if (c < N && (c >> 5) < a.words_stride) bm[c >> 5] = klo;
      if (c + 32 < N && (c >> 5) + 1 < a.words_stride) bm[(c >> 5) + 1] = khi;
    }
  }
  Z = tw_wave_scan_u64(Z);
  A = tw_wave_scan_u64(A);
  __shared__ uint32_t wc[NW];
  __shared__ unsigned long long wz[NW], wa[NW];
  if (lane == 63) { wc[wave] = cnt; wz[wave] = Z; wa[wave] = A; }
  __syncthreads();
  if (tid == 0) {
    uint32_t t = 0;
    unsigned long long tz = 0, ta = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) { t += wc[w]; tz += wz[w]; ta += wa[w]; }
    if (t) atomicAdd(&a.kdef[(long long)bh * TW_CTR], t);
    if (tz) atomicAdd(&a.sums[(long long)bh * WS_SUMS], tz);
    if (ta) atomicAdd(&a.sums[(long long)bh * WS_SUMS + 1], ta);
  }
}

constexpr int WR_CAP = 64;
struct ResolveLds {
  unsigned long long histM[HP_NB];
  uint32_t histC[HP_NB];
  unsigned long long cand_mass[WR_CAP];
  uint32_t cand_key[WR_CAP];
  uint32_t red[16], red2[16];
  uint32_t n, T;
};
// Block-wide minimum of lo and maximum of hi over waves whose results are in red / red2 (every lane gets them).
template <int NW>
__device__ __forceinline__ void wide_min_max(const ResolveLds& L, int lane, uint32_t* lo, uint32_t* hi) {
  *lo = (uint32_t)__builtin_amdgcn_readfirstlane((int)~tw_row_max_u32(~L.red[lane & (NW - 1)]));
  *hi = (uint32_t)__builtin_amdgcn_readfirstlane((int)tw_row_max_u32(L.red2[lane & (NW - 1)]));
}

// Threshold among scores of ranks [rlo, rlo + 2^shift): the largest key whose upper set, with the mass A above the
// interval, reaches `target`.  The interval is narrowed 9 bits per round with a 512-bucket LDS histogram until at most
// 64 scores are left, and those are compared exactly on the scores' own bits; more than 64 scores of one rank are one
// tier, and an interval that holds one score value only, however often, needs no narrowing.  each(f) calls f(key, score) for every score of this thread; called by all NT threads.  *found: the interval
// holds the crossing.
template <int NT, class Each>
__device__ __forceinline__ uint32_t wide_threshold(Each each, float m, uint32_t rlo, int shift, uint32_t pop, unsigned long long A,
                                                   unsigned long long target, ResolveLds& L, bool* found) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  *found = false;
  if (tid == 0) L.n = 0;
#pragma unroll 1
  for (bool first = true; pop > (uint32_t)WR_CAP && (shift > 0 || first); first = false) {
    const int nshift = shift >= 9 ? shift - 9 : 0;
    const uint32_t nb = 1u << (shift - nshift);   // buckets that cover the interval
    __syncthreads();
    for (int i = tid; i < HP_NB; i += NT) { L.histM[i] = 0; L.histC[i] = 0; }
    __syncthreads();
    // A thread's consecutive scores of one bucket are added up before they go to LDS (rows of equal keys put all their
    // scores into one bucket: 131072 of them 135 us a pass when each was added by itself).
    uint32_t cb = 0, cc = 0, klo = 0xFFFFFFFFu, khi = 0u;
    unsigned long long cm = 0;
    auto flush = [&]() {
      if (cc) { atomicAdd(&L.histM[cb], cm); atomicAdd(&L.histC[cb], cc); }
    };
    each([&](uint32_t k, float s) {
      const uint32_t r = hp_rank_only(m, s);
      const uint32_t bk = (r - rlo) >> nshift;
      if (r != HP_NONE && r >= rlo && bk < nb) {
        klo = k < klo ? k : klo;
        khi = k > khi ? k : khi;
        if (bk != cb) { flush(); cb = bk; cm = 0; cc = 0; }
        cm += hp_fix(hp_numer(m, s));
        cc += 1;
      }
    });
    flush();
    klo = ~tw_wave_max_u32(~klo);
    khi = tw_wave_max_u32(khi);
    if (lane == 0) { L.red[wave] = klo; L.red2[wave] = khi; }
    __syncthreads();
    wide_min_max<NT / 64>(L, lane, &klo, &khi);
    unsigned long long mb[8], mine = 0;           // every wave scans on its own: lane l owns buckets 8l .. 8l+7
#pragma unroll
    for (int k = 0; k < 8; ++k) { mb[k] = L.histM[8 * lane + k]; mine += mb[k]; }
    const unsigned long long incl = tw_wave_scan_u64(mine);
    const unsigned long long before = A + incl - mine;
    const bool hit = before < target && before + mine >= target;
    const unsigned long long bal = __ballot(hit);
    if (bal == 0) return 0xFFFFFFFFu;             // (the same in every wave)
    if (klo == khi) { *found = true; return klo; }
    const int src = __ffsll((long long)bal) - 1;
    unsigned long long cum = before, asel = before;
    int bsel = 0;
#pragma unroll
    for (int k = 0; k < 8; ++k) {
      if (cum < target && cum + mb[k] >= target) { bsel = k; asel = cum; }
      cum += mb[k];
    }
    const int bucket = 8 * src + __shfl(bsel, src, 64);
    A = __shfl(asel, src, 64);
    pop = L.histC[bucket];
    rlo += (uint32_t)bucket << nshift;
    shift = nshift;
  }
  const uint32_t rhi = rlo + (1u << shift) - 1u;
  const bool small = pop <= (uint32_t)WR_CAP;
  uint32_t kmin = 0xFFFFFFFFu;
  __syncthreads();                                // L.n cleared; scans done
  each([&](uint32_t k, float s) {
    const uint32_t r = hp_rank_only(m, s);
    if (r != HP_NONE && r >= rlo && r <= rhi) {
      kmin = k < kmin ? k : kmin;
      if (small) {
        const uint32_t at = atomicAdd(&L.n, 1u);
        if (at < (uint32_t)WR_CAP) { L.cand_key[at] = k; L.cand_mass[at] = hp_fix(hp_numer(m, s)); }
      }
    }
  });
  if (!small) {                                   // more than WR_CAP scores of one rank: keep them all
    kmin = ~tw_wave_max_u32(~kmin);
    if (lane == 0) L.red[wave] = kmin;
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t T;
    if (small) {
      const uint32_t n = L.n < (uint32_t)WR_CAP ? L.n : (uint32_t)WR_CAP;
      const uint32_t kx = lane < (int)n ? L.cand_key[lane] : 0u;
      unsigned long long S = 0;
#pragma unroll 4
      for (uint32_t j = 0; j < n; ++j) S += L.cand_key[j] >= kx ? L.cand_mass[j] : 0ull;
      const uint32_t best = (lane < (int)n && A + S >= target) ? kx : 0u;
      T = tw_wave_max_u32(best);
    } else {
      T = L.red[0];
#pragma unroll
      for (int w = 1; w < NT / 64; ++w) T = L.red[w] < T ? L.red[w] : T;
    }
    if (lane == 0) L.T = T;
  }
  __syncthreads();
  const uint32_t T = L.T;
  *found = T != 0u && A < target;
  return *found ? T : 0xFFFFFFFFu;
}

// One workgroup per head walks the head's list (a few dozen scores as a rule, some thousand in a near-uniform row).  A
// head whose list overflowed or does not hold the threshold (the exact sums decide) is searched from its whole row
// instead, and its bitmap written anew: one to three narrowing passes over the row (one where the undecided scores are
// all equal), the exact one and the bitmap's, bound by one workgroup's loads in flight.  Whole top-p of such rows:
// 256 heads x 262144 equal keys 198 us (ordinary keys 85), logits within 0.01 of each other 187, keys drawn from four
// rows 264; 32 heads x 131072 75 / 31 (the list holds them) / 68 (ordinary keys 26).
template <int NT>
__global__ __launch_bounds__(NT) void wide_resolve_kernel(WideArgs a) {
  constexpr int NW = NT / 64;
  const int bh = blockIdx.x, b = bh / a.Hq, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  __shared__ ResolveLds L;
  const uint2* const list = a.ulist + (long long)bh * W_CAP;
  const uint2 first = list[tid];                  // (inside the buffer whatever the list's length; all loads of the prologue together)
  const uint32_t listed = (uint32_t)__builtin_amdgcn_readfirstlane((int)a.ucount[(long long)bh * TW_CTR]);
  const unsigned long long Z0 = a.sums[(long long)bh * WS_SUMS], A0 = a.sums[(long long)bh * WS_SUMS + 1];
  const uint32_t mk = wide_headmax(a.headmax, bh, lane);
  const bool search = !a.keep_all && mk != 0;
  const float m = tw_key_to_float(mk);
  uint32_t* const bm = a.bitmaps + (long long)bh * a.words_stride;
  uint32_t add = 0;
  bool whole_row = false;
  if (search) {                                   // block-uniform
    const uint32_t cn = listed < (uint32_t)W_CAP ? listed : (uint32_t)W_CAP;
    auto walk = [&](auto f) {                     // f(key, token); the first NT entries sit in registers
      if ((uint32_t)tid < cn) f(first.x, first.y);
#pragma unroll 4
      for (uint32_t i = (uint32_t)(NT + tid); i < cn; i += NT) { const uint2 x = list[i]; f(x.x, x.y); }
    };
    uint32_t T = 0xFFFFFFFFu;
    bool found = false;
    const unsigned long long target = hp_target(a.p, Z0);
    if (listed > 0 && listed <= (uint32_t)W_CAP && A0 < target) {           // block-uniform
      uint32_t rlo = 0;
      int shift = 0;
      if (cn > (uint32_t)WR_CAP) {                // ranks the list spans (a short one is resolved as it is: 27 bits hold every rank)
        uint32_t rmin = 0xFFFFFFFFu, rmax = 0u;
        walk([&](uint32_t k, uint32_t) {
          const uint32_t r = hp_rank_only(m, tw_key_to_float(k));
          rmin = r < rmin ? r : rmin;
          rmax = r > rmax ? r : rmax;
        });
        rmin = ~tw_wave_max_u32(~rmin);
        rmax = tw_wave_max_u32(rmax);
        if (lane == 0) { L.red[wave] = rmin; L.red2[wave] = rmax; }
        __syncthreads();
        wide_min_max<NW>(L, lane, &rlo, &rmax);
        const uint32_t span = rmax - rlo;
        shift = span ? 32 - __clz(span) : 0;
      } else {
        shift = 27;
      }
      auto each = [&](auto f) { walk([&](uint32_t k, uint32_t) { f(k, tw_key_to_float(k)); }); };
      T = wide_threshold<NT>(each, m, rlo, shift, cn, A0, target, L, &found);
    }
    if (found) {
      walk([&](uint32_t k, uint32_t t) {
        if (k >= T && (t >> 5) < (uint32_t)a.words_stride) {
          atomicOr(&bm[t >> 5], 1u << (t & 31));
          add += 1;
        }
      });
    }
    whole_row = !found;
  }
  if (whole_row) {                                // block-uniform
    const int count = wide_count(a, b, bh);
    const int N = count * TW_PAGE;
    const float* row = a.scores + (long long)bh * a.cand_stride;
    auto each = [&](auto f) {
#pragma unroll 1
      for (int c0 = tid * 4; c0 < N; c0 += 16 * NT) {                        // four loads in flight per thread
        float4 x[4];
#pragma unroll
        for (int v = 0; v < 4; ++v) x[v] = *(const float4*)(row + (c0 + v * 4 * NT < N ? c0 + v * 4 * NT : N - 4));
#pragma unroll
        for (int v = 0; v < 4; ++v) {
          if (c0 + v * 4 * NT < N) {
            const float y[4] = {x[v].x, x[v].y, x[v].z, x[v].w};
#pragma unroll
            for (int k = 0; k < 4; ++k) f(tw_float_key(y[k]), y[k]);
          }
        }
      }
    };
    // first among the ranks that the histogram left undecided (an overflowed list), then - the sums say that the
    // threshold is not there - among all
    const unsigned long long target = hp_target(a.p, Z0);
    uint32_t T = 0xFFFFFFFFu;
    bool found = false;
    if (A0 < target) {                              // block-uniform
      const float4 rg = a.range[bh];
      const uint32_t rlo = (uint32_t)(rg.y * 4194304.f), span = (uint32_t)(rg.z * 4194304.f) - rlo;   // (rg.y < rg.z <= 27.5)
      T = wide_threshold<NT>(each, m, rlo, span > 1u ? 32 - __clz(span - 1u) : 0, 0xFFFFFFFFu, A0, target, L, &found);
    }
    if (!found) T = wide_threshold<NT>(each, m, 0u, 27, 0xFFFFFFFFu, 0ull, target, L, &found);
    // 16 slots = one page = one half word of the bitmap per thread
    for (int i = tid; i < count; i += NT) {
      uint32_t bits = 0;
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const float4 x = *(const float4*)(row + i * 16 + 4 * v);
        const float y[4] = {x.x, x.y, x.z, x.w};
#pragma unroll
        for (int k = 0; k < 4; ++k)
          bits |= (hp_rank_only(m, y[k]) != HP_NONE && tw_float_key(y[k]) >= T ? 1u : 0u) << (4 * v + k);
      }
      const int pgi = a.sel_pages ? a.sel_pages[(long long)bh * a.max_sel + i] : i;
      if (pgi >= 0 && (pgi >> 1) < a.words_stride) ((unsigned short*)bm)[pgi] = (unsigned short)bits;
      add += __popc(bits);
    }
  }
  add = tw_wave_scan_u32(add);
  __syncthreads();                                // red is reused
  if (lane == 63) L.red[wave] = add;
  __syncthreads();
  if (tid == 0) {
    uint32_t t = whole_row ? 0u : a.kdef[(long long)bh * TW_CTR];
    for (int w = 0; w < NW; ++w) t += L.red[w];
    a.kept_count[bh] = (int32_t)t;
  }
}

struct ListArgs {
  const uint32_t* bitmaps;
  const int32_t* seq_lens;
  int32_t* count_out;         // or nullptr (count already known)
  int32_t* idx_out;
  uint32_t* status;
  int rows_per_seq, maps_per_row, max_pages, words_stride, out_stride;
  uint32_t trunc_bit;
  uint32_t* segcnt;           // [row][segs]: set bits per segment, filled by bitmap_count_kernel; nullptr = count in place
  int segs;
};

// Row r: OR of NB consecutive bitmaps (r * maps_per_row ...) -> ascending positions.  One
// workgroup per (segment of 256 words, row): its output offset is the number of bits in the
// row's earlier segments - read from the per-segment counts that bitmap_count_kernel left
// (long rows), or counted in place (rows of a few segments); it then stages its own positions
// in LDS and copies them out coalesced.  The workgroup of the last segment also writes the count.
constexpr int BL_SEG = 256;
__device__ __forceinline__ int list_words(const ListArgs& a, int row) {
  const int n = a.seq_lens[row / a.rows_per_seq];
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  const int ntok = P * TW_PAGE < n ? P * TW_PAGE : n;
  return (ntok + 31) >> 5;
}
template <int NB>
__global__ __launch_bounds__(256) void bitmap_count_kernel(ListArgs a) {
  const int row = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x;
  const int nwords = list_words(a, row);            // (words beyond the sequence's end were never written)
  const uint32_t* bm = a.bitmaps + (long long)row * a.maps_per_row * a.words_stride;
  const int wi = seg * BL_SEG + tid;
  uint32_t w = 0;
  if (wi < nwords) {
#pragma unroll
    for (int hh = 0; hh < NB; ++hh) w |= bm[(long long)hh * a.words_stride + wi];
  }
  __shared__ uint32_t ws32[16];
  uint32_t total;
  tw_block_scan_u32(__popc(w), ws32, &total);
  if (tid == 0) a.segcnt[(long long)row * a.segs + seg] = total;
}

template <int NB>
__global__ __launch_bounds__(256) void bitmap_list_kernel(ListArgs a) {
  const int row = blockIdx.y, seg = blockIdx.x, tid = threadIdx.x;
  const int nwords = list_words(a, row);
  const int nseg = (nwords + BL_SEG - 1) / BL_SEG;
  if (seg >= nseg && !(seg == 0 && nseg == 0)) return;
  __shared__ uint32_t ws32[16];
  __shared__ int32_t stage[BL_SEG * 32];
  const uint32_t* bm = a.bitmaps + (long long)row * a.maps_per_row * a.words_stride;
  int32_t* out = a.idx_out + (long long)row * a.out_stride;
  // bits before this segment
  uint32_t before = 0;
  if (a.segcnt) {
    for (int s0 = tid; s0 < seg; s0 += 256) before += a.segcnt[(long long)row * a.segs + s0];
  } else
  for (int s0 = 0; s0 < seg; s0 += 4) {             // 4 clamped loads in flight
    uint32_t x[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool ok = s0 + j < seg;
      const int wi = ok ? (s0 + j) * BL_SEG + tid : 0;
      uint32_t v = 0;
#pragma unroll
      for (int hh = 0; hh < NB; ++hh) v |= bm[(long long)hh * a.words_stride + wi];
      x[j] = ok ? v : 0u;
    }
    before += __popc(x[0]) + __popc(x[1]) + __popc(x[2]) + __popc(x[3]);
  }
  const int wi = seg * BL_SEG + tid;
  uint32_t w = 0;
  if (wi < nwords) {
#pragma unroll
    for (int hh = 0; hh < NB; ++hh) w |= bm[(long long)hh * a.words_stride + wi];
  }
  uint32_t base_total, total;
  tw_block_scan_u32(before, ws32, &base_total);
  const uint32_t incl = tw_block_scan_u32(__popc(w), ws32, &total);
  uint32_t pos = incl - __popc(w);
  while (w) {
    const int bit = __ffs(w) - 1;
    w &= w - 1;
    stage[pos++] = wi * 32 + bit;
  }
  __syncthreads();
  for (uint32_t i = tid; i < total; i += 256)
    if (base_total + i < (uint32_t)a.out_stride) out[base_total + i] = stage[i];
  if (tid == 0 && seg == (nseg > 0 ? nseg - 1 : 0)) {
    uint32_t run = base_total + total;
    if (run > (uint32_t)a.out_stride) { atomicOr(a.status, a.trunc_bit); run = a.out_stride; }
    if (a.count_out) a.count_out[row] = (int32_t)run;
  }
}

template <int NB>
int launch_list(ListArgs a, int rows, uint32_t* segcnt, hipStream_t s) {
  int err = TW_OK;
  const int max_words = (a.max_pages + 1) / 2;
  int segs = (max_words + BL_SEG - 1) / BL_SEG;
  if (segs < 1) segs = 1;
  a.segs = segs;
  a.segcnt = segs > 4 ? segcnt : nullptr;           // few segments: counting the earlier ones in place is cheaper than a launch
  if (a.segcnt) {                                    // a launch of its own: close the caller's bracket, open another
    TW_LAUNCH(bitmap_count_kernel<NB>, dim3(segs, rows), dim3(256), 0, s, a);
    err = tw_prof_after(s);
    tw_prof_before(TW_K_UNION, s);
  }
  TW_LAUNCH(bitmap_list_kernel<NB>, dim3(segs, rows), dim3(256), 0, s, a);
  return err;
}

}  // namespace

// Everything after the scores have been written (headmax filled by the scoring kernel; hist_done: the mass histogram
// too).  tw_prune_wide_init must have been enqueued BEFORE the scoring kernel.
int tw_prune_wide_init(const PruneWs& L, void* ws, bool full, hipStream_t s) {
  // every token a candidate: every bitmap word inside a sequence is written, the bitmaps need no clearing
  const size_t n16 = ((full ? L.bitmaps : L.grid) - L.headmax) / 16;
  tw_prof_before(TW_K_TOPP, s);
  TW_LAUNCH(wide_init_kernel, dim3((unsigned)((n16 + 255) / 256)), dim3(256), 0, s, (uint4*)((char*)ws + L.headmax), n16);
  return tw_prof_after(s);
}

int tw_prune_wide(const TwDims& d, const PruneWs& L, void* ws, const twilight_kv_t* kv, const int32_t* sel_pages,
                  const int32_t* sel_count, int max_sel, int cand_stride, float p, int32_t* kept_count,
                  int32_t* kept_idx, int kept_stride, int32_t* union_count, int32_t* union_idx, int union_stride,
                  uint32_t* status, bool hist_done, hipStream_t s) {
  char* base = (char*)ws;
  WideArgs a;
  a.scores = (const float*)(base + L.scores); a.sel_pages = sel_pages; a.sel_count = sel_count; a.seq_lens = kv->seq_lens;
  a.headmax = (const uint32_t*)(base + L.headmax); a.ghist = (unsigned long long*)(base + L.ghist); a.hgrid = (WhGrid*)(base + L.grid);
  a.range = (float4*)(base + L.range);
  a.sums = (unsigned long long*)(base + L.sums);
  a.ulist = (uint2*)(base + L.ulist);
  a.ucount = (uint32_t*)(base + L.ucount); a.kdef = (uint32_t*)(base + L.kdef);
  a.bitmaps = (uint32_t*)(base + L.bitmaps); a.kept_count = kept_count; a.status = status;
  a.Hq = d.Hq; a.max_pages = d.max_pages; a.max_sel = max_sel; a.cand_stride = cand_stride;
  a.words_stride = L.words_stride; a.keep_all = p >= 1.0f ? 1 : 0; a.p = p;
  const int nbh = d.batch * d.Hq;
  // histogram pass: large workgroups (fewer flushes of the LDS histogram per score) unless a row fits a small one; emit pass: small ones (they
  // overlap their load and compute phases)
  constexpr int HIST_NT = 1024, EMIT_NT = 256;
  auto grid_for = [&](int nt) { return dim3((cand_stride + nt * W_SLOTS - 1) / (nt * W_SLOTS), nbh); };
  if (!a.keep_all && !hist_done) {
    tw_prof_before(TW_K_TOPP, s);
    if (cand_stride <= 256 * W_SLOTS) TW_LAUNCH(wide_hist_kernel<256>, grid_for(256), dim3(256), 0, s, a);
    else TW_LAUNCH(wide_hist_kernel<HIST_NT>, grid_for(HIST_NT), dim3(HIST_NT), 0, s, a);
    if (int e = tw_prof_after(s)) return e;
  }
  if (!a.keep_all) {
    tw_prof_before(TW_K_TOPP, s);
    TW_LAUNCH(wide_decide_kernel, dim3(nbh), dim3(64), 0, s, a);
    if (int e = tw_prof_after(s)) return e;
  }
  tw_prof_before(TW_K_TOPP, s);
  TW_LAUNCH(wide_emit_kernel<EMIT_NT>, grid_for(EMIT_NT), dim3(EMIT_NT), 0, s, a);
  if (int e = tw_prof_after(s)) return e;
  tw_prof_before(TW_K_TOPP, s);
  // one 1024-thread workgroup fits a CU; more heads than CUs share them better in small ones
  if (nbh > tw_num_cus()) TW_LAUNCH(wide_resolve_kernel<256>, dim3(nbh), dim3(256), 0, s, a);
  else TW_LAUNCH(wide_resolve_kernel<1024>, dim3(nbh), dim3(1024), 0, s, a);
  if (int e = tw_prof_after(s)) return e;

  uint32_t* segcnt = (uint32_t*)(base + L.segcnt);
  ListArgs l;
  l.bitmaps = a.bitmaps; l.seq_lens = kv->seq_lens; l.status = status; l.max_pages = d.max_pages;
  l.words_stride = L.words_stride;
  if (kept_idx) {
    l.count_out = kept_count; l.idx_out = kept_idx; l.rows_per_seq = d.Hq; l.maps_per_row = 1; l.out_stride = kept_stride;
    l.trunc_bit = TW_STATUS_KEPT_TRUNCATED;
    tw_prof_before(TW_K_UNION, s);
    const int le = launch_list<1>(l, nbh, segcnt, s);
    if (int e = tw_prof_after(s)) return e;
    if (le) return le;
  }
  l.count_out = union_count; l.idx_out = union_idx; l.rows_per_seq = d.Hkv; l.maps_per_row = d.G; l.out_stride = union_stride;
  l.trunc_bit = TW_STATUS_UNION_TRUNCATED;
  tw_prof_before(TW_K_UNION, s);
  int le;
  switch (d.G) {
    case 1: le = launch_list<1>(l, d.batch * d.Hkv, segcnt, s); break;
    case 2: le = launch_list<2>(l, d.batch * d.Hkv, segcnt, s); break;
    case 4: le = launch_list<4>(l, d.batch * d.Hkv, segcnt, s); break;
    default: le = launch_list<8>(l, d.batch * d.Hkv, segcnt, s); break;
  }
  if (int e = tw_prof_after(s)) return e;
  return le;
}
