// Stage 2: the Twilight pruner (paper: Section 4.2, Algorithm 1,
// Definition 3.3, Appendix B.1 and B.2).
//
// int4_score       estimated logits from the quantised K copy.  One wave = one
//                  page per step: 64 lanes x 16 B = the page's 1 KiB of codes,
//                  lane = (token, group of 32 dims); 8 integer products of 4
//                  or, 4-bit codes of one head per page, 8 values per lane and
//                  head, scale/zero applied per group, quad DPP sum over the
//                  4 groups.  Templated on the code width (2 / 4 / 8 bits).
// int4_score_mfma  the same scores on the matrix cores, used when every page
//                  is a candidate and 4 or 8 query heads share each page.
// topp_head        per (sequence, query head), scores in registers: max, then
//                  a mass histogram over the fixed-point distance to the max
//                  logit narrows the threshold 9 bits per pass (masses in
//                  64-bit fixed point, so sums do not depend on the order of
//                  the atomics), finished by an exact resolve on the scores'
//                  own bit patterns inside one wave.  Kept tokens go to a
//                  bitmap; the last head of a KV group to finish ORs the
//                  group's bitmaps into the sorted union list.
// Rows too long for registers take the multi-workgroup path in topp_wide.hip.
#include <stdlib.h>
#include "topp_common.h"
#include "select_body.h"

namespace {

constexpr float kInv127 = 0x1.020408p-7f;    // fp32(1/127)
constexpr float kRsqrtD = 0x1.6a09e6p-4f;    // fp32(1/sqrt(128))
constexpr float kLog2e = 0x1.715476p+0f;

// ------------------------------------------------------------------ int4_score
struct ScoreArgs {
  const uint16_t* q;          // bf16 [b][Hq][128]
  const int32_t* sel_pages;   // [b][Hq][max_sel] or nullptr (all pages)
  const int32_t* sel_count;
  const int32_t* page_table;
  const int32_t* seq_lens;
  const uint4* kq_pool;       // 64 uint4 per (page, head)
  const uint32_t* kq_meta;    // 64 words per (page, head)
  float* scores;              // [b][Hq][cand_stride]
  int32_t* dots;              // [b][Hq][cand_stride][4] or nullptr
  uint32_t* arrive;           // [b][Hkv] arrival counters of the top-p kernel that follows, or nullptr
  uint32_t* headmax;          // [b][Hq][HM_SLOTS] keys whose maximum is the head's largest score (atomicMax), or nullptr
  unsigned long long* ghist;  // [b][Hq][WH_NB] histograms, added to (HIST kernels) ...
  const WhGrid* hgrid;        // ... over the grids [b][Hq]
  const uint32_t* chmask;     // [Hkv][4] channels of the query that take part (bit d % 32 of word d / 32), or nullptr = all
  int Hq, Hkv, max_pages, max_sel, cand_stride, pw;   // pw: pages per wave (<= 64)
  int rotate;                 // list mode with a grid a multiple of 8 wide: chunk = (column - group % 8) mod width
  long long pool_pages;
};

// q of NH consecutive heads -> int8 (symmetric per head: sq = max|q| * (1/127), round half even),
// 4 values per word, and c = sq / sqrt(128) per head.  Called by all threads of the block; wave w takes the heads w,
// w + waves, ..., two values per lane, with all of its loads out first (one head after the other by the whole block, each
// with its load and two barriers, kept every workgroup of an 8-head scoring launch about 5 us from its first page).
// chmask: 4 words of the KV head's channel set, or nullptr - channels outside it get the int8 value 0 (the scale sq
// is that of the whole query), which restricts the estimate to the set (channel-sparse token selector).
template <int NH, int NT = 256>
__device__ __forceinline__ void tw_quantize_q(const uint16_t* q, int (*qi_s)[32], float* c_s, const uint32_t* chmask = nullptr) {
  constexpr int NW = NT / 64, R = (NH + NW - 1) / NW;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  uint32_t raw[R];
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int h = wave + r * NW < NH ? wave + r * NW : NH - 1;
    __builtin_memcpy(&raw[r], q + (h * 64 + lane) * 2, 4);     // (bf16 rows may begin at any element: no more than 2-byte alignment)
  }
  const uint32_t cm = chmask ? chmask[lane >> 4] >> ((2 * lane) & 31) : 3u;
#pragma unroll
  for (int r = 0; r < R; ++r) {
    const int h = wave + r * NW;
    const float v[2] = {tw_bf16_lo(raw[r]), tw_bf16_hi(raw[r])};
    const float sq = __fmul_rn(tw_wave_max_f(fmaxf(fabsf(v[0]), fabsf(v[1]))), kInv127);
    uint32_t bytes = 0;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      int qi = 0;
      if (sq > 0.f) {
        float t = rintf(__fdiv_rn(v[i], sq));
        t = fminf(fmaxf(t, -127.f), 127.f);
        qi = (int)t;
      }
      if (!((cm >> i) & 1u)) qi = 0;
      bytes |= ((uint32_t)qi & 0xFFu) << (8 * i);
    }
    if (h < NH) {                                  // wave-uniform
      ((uint16_t*)qi_s[h])[lane] = (uint16_t)bytes;
      if (lane == 0) c_s[h] = __fmul_rn(sq, kRsqrtD);
    }
  }
  __syncthreads();
}

// The same for one head by every wave on its own, without a barrier: raw = the lane's pair of bf16 values, qi = 32 words of LDS that
// are the wave's.  Returns c.
__device__ __forceinline__ float tw_quantize_q1(uint32_t raw, int* qi) {
  const int lane = threadIdx.x & 63;
  const float v[2] = {tw_bf16_lo(raw), tw_bf16_hi(raw)};
  const float sq = __fmul_rn(tw_wave_max_f(fmaxf(fabsf(v[0]), fabsf(v[1]))), kInv127);
  uint32_t bytes = 0;
  if (sq > 0.f) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float t = rintf(__fdiv_rn(v[i], sq));
      t = fminf(fmaxf(t, -127.f), 127.f);
      bytes |= ((uint32_t)(int)t & 0xFFu) << (8 * i);
    }
  }
  ((uint16_t*)qi)[lane] = (uint16_t)bytes;
  asm volatile("" ::: "memory");                   // (a wave's LDS accesses are done in order)
  return __fmul_rn(sq, kRsqrtD);
}

// One lane's group of 32 codes of slot (token, group) `idx` of the pool, as stored.
// STREAM: the codes are read once (every page a candidate, all heads of the group in one workgroup) and loaded
// non-temporally; with per-head page lists they stay cached for the other heads of the group.
template <int BITS, bool STREAM = false>
__device__ __forceinline__ void tw_load_raw(const uint4* kq_pool, long long idx, uint4 (&r)[BITS == 8 ? 2 : 1]) {
  if (BITS == 4) r[0] = STREAM ? tw_ld_stream(kq_pool + idx) : kq_pool[idx];
  else if (BITS == 2) { const uint2 c = ((const uint2*)kq_pool)[idx]; r[0] = make_uint4(c.x, c.y, 0u, 0u); }
  else { r[0] = kq_pool[idx * 2]; r[BITS == 8 ? 1 : 0] = kq_pool[idx * 2 + 1]; }
}
// A whole page's codes and (scale, zero) words by a wave, the page (row = pool page * Hkv + KV head) the same for all lanes: as
// buffers of the page's own size, so that the addresses are scalar and a page that is not there reads as zeros without going to memory.
// (What bounds many heads' scoring is vector instructions, next to the phases' barriers: 35 per page and wave with 64-bit vector
// addresses, a validity test per token and (scale, zero) words converted before they were multiplied, 22 so.  The one-launch
// selector + pruner, us: 5 x 64 heads x 5960 candidates 40.8 -> 36.6, 48 ragged sequences x 32 heads of up to 5000 51.9 -> 45.0,
// 64 of up to 8192 100.5 -> 95.5, 1024 x 4096 55.9 -> 54.2, 8 x 32 x 4096 21.1 -> 20.7.)
template <int BITS>
__device__ __forceinline__ void tw_load_page(const uint4* kq_pool, const uint32_t* kq_meta, long long row, bool there, int lane,
                                             uint4 (&r)[BITS == 8 ? 2 : 1], uint32_t* meta) {
  constexpr int BYTES = 256 * BITS, FORMAT = 0x00027000;
  const auto codes = __builtin_amdgcn_make_buffer_rsrc((char*)kq_pool + row * BYTES, 0, there ? BYTES : 0, FORMAT);
  const auto words = __builtin_amdgcn_make_buffer_rsrc((char*)kq_meta + row * 256, 0, there ? 256 : 0, FORMAT);
  if (BITS == 2) {
    const auto c = __builtin_amdgcn_raw_buffer_load_b64(codes, lane * 8, 0, 0);
    r[0] = make_uint4(c[0], c[1], 0u, 0u);
  } else {
#pragma unroll
    for (int i = 0; i < (BITS == 8 ? 2 : 1); ++i) {
      const auto c = __builtin_amdgcn_raw_buffer_load_b128(codes, lane * (4 * BITS) + 16 * i, 0, 0);
      r[i] = make_uint4(c[0], c[1], c[2], c[3]);
    }
  }
  *meta = __builtin_amdgcn_raw_buffer_load_b32(words, lane * 4, 0, 0);
}
// One lane's query words: q8 = its group's 8 words of 4 int8 values (dims 8w .. 8w+3, then 8w+4 .. 8w+7).  4-bit codes meet
// them as they are stored, 8 to a word, byte k = code[k] | code[k+4] << 4: a query value is 16 * high + low with low an unsigned and high a
// signed 4-bit number, one product sum each (the codes minus 8 are signed 4-bit numbers, their bits but for the top one of each).
// Unpacked to bytes for 4-value products a page takes 7 vector instructions more: 12 unpack, where 4 flip the top bits and one adds the
// halves.  The one-launch selector + pruner, us: 512 heads x 8192 candidates 55.3 -> 51.9, 64 ragged sequences x 32 heads of up to 8192
// 135.4 -> 128.2, 1024 heads x 4096 52.4 -> 50.8; steps gain 1 % and less.
// Not SPLIT (int4_score_kernel with two and more heads per loaded page, which share the codes once unpacked): 4-value products.  A wave's
// few pages do not pay back the making of several heads' split words, and the registers cost a wave per SIMD (2 heads, dots stored: 66
// for 64).  Two heads per KV head, us, split / not: 8 x 32 heads x 32768 tokens with dots 89.5 / 83.0 and without 69.6 / 69.8, without
// dots 3 x 32 x 9001 9.25 / 8.98, 4 x 8 x 16384 5.58 / 5.37.
// *qs = sum of the values, *i0 = where the group's sum starts.
template <int BITS, bool SPLIT = BITS == 4>
__device__ __forceinline__ void tw_query_words(const int* q8, int (&qw)[8], int* qs, int* i0) {
  int sum = 0;
#pragma unroll
  for (int k = 0; k < 8; ++k) {
    qw[k] = q8[k];
    sum = __builtin_amdgcn_sdot4(qw[k], 0x01010101, sum, false);
  }
  *qs = sum;
  *i0 = BITS == 8 ? 128 * sum : 0;                // 8-bit codes enter the signed product as code - 128
  if (SPLIT) {
    int high[4], low[4], hs = 0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const uint32_t x = (uint32_t)qw[2 * w], y = (uint32_t)qw[2 * w + 1];
      low[w] = (int)((x & 0x0F0F0F0Fu) | ((y & 0x0F0F0F0Fu) << 4));
      high[w] = (int)(((x >> 4) & 0x0F0F0F0Fu) | (y & 0xF0F0F0F0u));
      hs = __builtin_amdgcn_sdot8(high[w], 0x11111111, hs, false);
    }
#pragma unroll
    for (int w = 0; w < 4; ++w) { qw[w] = high[w]; qw[4 + w] = low[w]; }
    *i0 = 128 * hs;
  }
}
// I = sum over the group's 32 dims of q * code
template <int BITS, bool SPLIT = BITS == 4>
__device__ __forceinline__ int tw_group_dot(const int (&qw)[8], const uint4 (&r)[BITS == 8 ? 2 : 1], int i0) {
  if (SPLIT) {
    const uint32_t wv[4] = {r[0].x, r[0].y, r[0].z, r[0].w};
    int h = 0;
    uint32_t l = (uint32_t)i0;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      h = __builtin_amdgcn_sdot8(qw[w], (int)(wv[w] ^ 0x88888888u), h, false);
      l = __builtin_amdgcn_udot8((uint32_t)qw[4 + w], wv[w], l, false);
    }
    return (int)(((uint32_t)h << 4) + l);
  }
  int u[8];
  if (BITS == 4) {
    u[0] = r[0].x & 0x0F0F0F0F; u[1] = (r[0].x >> 4) & 0x0F0F0F0F;
    u[2] = r[0].y & 0x0F0F0F0F; u[3] = (r[0].y >> 4) & 0x0F0F0F0F;
    u[4] = r[0].z & 0x0F0F0F0F; u[5] = (r[0].z >> 4) & 0x0F0F0F0F;
    u[6] = r[0].w & 0x0F0F0F0F; u[7] = (r[0].w >> 4) & 0x0F0F0F0F;
  } else if (BITS == 2) {
    u[0] = r[0].x & 0x03030303; u[1] = (r[0].x >> 2) & 0x03030303; u[2] = (r[0].x >> 4) & 0x03030303; u[3] = (r[0].x >> 6) & 0x03030303;
    u[4] = r[0].y & 0x03030303; u[5] = (r[0].y >> 2) & 0x03030303; u[6] = (r[0].y >> 4) & 0x03030303; u[7] = (r[0].y >> 6) & 0x03030303;
  } else {
    constexpr int H = BITS == 8 ? 1 : 0;
    u[0] = r[0].x ^ 0x80808080; u[1] = r[0].y ^ 0x80808080; u[2] = r[0].z ^ 0x80808080; u[3] = r[0].w ^ 0x80808080;
    u[4] = r[H].x ^ 0x80808080; u[5] = r[H].y ^ 0x80808080; u[6] = r[H].z ^ 0x80808080; u[7] = r[H].w ^ 0x80808080;
  }
  int I = i0;
#pragma unroll
  for (int k = 0; k < 8; ++k) I = __builtin_amdgcn_sdot4(qw[k], u[k], I, false);
  return I;
}
// the group's term of the score: fl(scale * I) + fl(zero * sum q), summed over the 4 groups of the
// token (the 4 lanes of a quad) in the fixed order (T0 + T1) + (T2 + T3).  MIX: the half-precision factors are taken as they lie in
// their word, each product rounded as it is by an fma with -0: for the head kernel's scoring loop, which vector instructions bound.  (The
// scoring launches wait for memory and gain nothing: token lists of 4 x 32 heads 4.65 us, 4.9 with it, of 10 x 32 6.25 and 6.3.)
template <bool MIX = false>
__device__ __forceinline__ float tw_token_sum(uint32_t meta, int I, float qsf) {
  float sI, zq;
  if (MIX) {
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel_hi:[1,0,0]" : "=v"(sI) : "v"(meta), "v"((float)I), "s"(0x80000000u));
    asm("v_fma_mix_f32 %0, %1, %2, %3 op_sel:[1,0,0] op_sel_hi:[1,0,0]" : "=v"(zq) : "v"(meta), "v"(qsf), "s"(0x80000000u));
  } else {
    sI = __fmul_rn(__half2float(__ushort_as_half((unsigned short)(meta & 0xFFFFu))), (float)I);
    zq = __fmul_rn(__half2float(__ushort_as_half((unsigned short)(meta >> 16))), qsf);
  }
  return tw_quad_sum(__fadd_rn(sI, zq));
}

// NH = heads scored per loaded page: 1 with per-head page lists, G when every
// page is a candidate (the G heads of a KV head then share each load).
template <int NH, bool FULL, bool DOTS, int UNR, int BITS = 4>
__global__ __launch_bounds__(256) void int4_score_kernel(ScoreArgs a) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int b, g, h0;
  if (FULL) { b = blockIdx.y / a.Hkv; g = blockIdx.y % a.Hkv; h0 = g * NH; }
  else      { b = blockIdx.y / a.Hq;  h0 = blockIdx.y % a.Hq; g = h0 / (a.Hq / a.Hkv); }
  const int n = a.seq_lens[b];
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  int count = P;
  if (!FULL) { count = a.sel_count[b * a.Hq + h0]; if (count > a.max_sel) count = a.max_sel; }
  // A workgroup takes the chunks of 4 * pw pages number blockIdx.x, blockIdx.x + gridDim.x, ... of its row
  // (one chunk each when the grid covers the row bound; fewer, looping workgroups for batches of many heads,
  // whose lists are often far shorter than the bound).
  // Workgroups go to the 8 XCDs round robin in dispatch order, so with a grid a multiple of 8 wide column x runs on XCD x % 8
  // and the heads of a KV head, which select largely the same pages, find each other's pages in that XCD's
  // L2.  Rotating the chunks by the group's number keeps that and spreads the first chunks of short lists
  // over all XCDs.
  const int col = (!FULL && a.rotate) ? (int)((blockIdx.x + gridDim.x - ((unsigned)(b * a.Hkv + g) & 7u)) % gridDim.x) : (int)blockIdx.x;
  int wg_first = col * 4 * a.pw;
  if (a.arrive && blockIdx.x == 0 && tid == 0) a.arrive[(b * a.Hkv + g) * TW_CTR] = 0;
  if (wg_first >= count) return;

  // ---- this wave's pages: lane k holds the k-th one (logical id, pool id).  The first chunk's are
  //      issued before the query is quantised, so that the two dependent loads overlap that prologue.
  int first = wg_first + wave * a.pw;
  int my_lp = -1, my_pool = -1;
  if (lane < a.pw && first + lane < count) {
    my_lp = FULL ? first + lane : a.sel_pages[((long long)(b * a.Hq + h0)) * a.max_sel + first + lane];
    if (my_lp >= 0 && my_lp < P) {
      const int pp = a.page_table[(long long)b * a.max_pages + my_lp];
      if (pp >= 0 && pp < a.pool_pages) my_pool = pp;
    }
  }
  int npages = count - first;
  if (npages > a.pw) npages = a.pw;

  // ---- quantise q of the NH heads to int8 (symmetric, per head)
  __shared__ int qi_s[NH][32];
  __shared__ float c_s[NH];
  tw_quantize_q<NH>(a.q + ((long long)(b * a.Hq + h0)) * 128, qi_s, c_s, a.chmask ? a.chmask + g * 4 : nullptr);
  constexpr bool SPLIT = BITS == 4 && NH == 1;
  const int j = lane & 3;                       // this lane's group of 32 dims
  int qw[NH][8], i0[NH];
  float qsf[NH], cc[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) {
    int qs;
    tw_query_words<BITS, SPLIT>(qi_s[h] + 8 * j, qw[h], &qs, &i0[h]);
    qsf[h] = (float)qs;
    cc[h] = c_s[h];
  }

  float hm[NH];
#pragma unroll
  for (int h = 0; h < NH; ++h) hm[h] = -__builtin_inff();
#pragma unroll 1
  for (;;) {
#pragma unroll 1
  for (int k0 = 0; k0 < npages; k0 += UNR) {
   // UNR pages per round: first all their loads (unconditional: an unmapped page or one past the wave's last reads
   // pool page 0 and is masked below), so that they are in flight together, then the arithmetic
   uint4 raw[UNR][BITS == 8 ? 2 : 1];
   uint32_t metas[UNR];
   int lps[UNR], pools[UNR];
#pragma unroll
   for (int kk = 0; kk < UNR; ++kk) {
    const int k = k0 + kk;                     // wave-uniform
    lps[kk] = __builtin_amdgcn_readlane(my_lp, k & 63);
    const int pl = __builtin_amdgcn_readlane(my_pool, k & 63);
    pools[kk] = k < npages ? pl : -1;
    const long long blk = ((long long)(pools[kk] >= 0 ? pools[kk] : 0) * a.Hkv + g) * 64;
    tw_load_raw<BITS, FULL>(a.kq_pool, blk + lane, raw[kk]);
    metas[kk] = FULL ? __builtin_nontemporal_load(a.kq_meta + blk + lane) : a.kq_meta[blk + lane];
   }
#pragma unroll
   for (int kk = 0; kk < UNR; ++kk) {
    const int k = k0 + kk;
    const int lp = lps[kk], pool = pools[kk];
    const uint32_t meta = metas[kk];
    const int tok = lp * TW_PAGE + (lane >> 2);
    const bool valid = pool >= 0 && tok < n;
    const long long slot = (long long)(first + k) * TW_PAGE + (lane >> 2);
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const int I = tw_group_dot<BITS, SPLIT>(qw[h], raw[kk], i0[h]);
      const float T = tw_token_sum(meta, I, qsf[h]);
      const float s = valid ? __fmul_rn(T, cc[h]) : -__builtin_inff();
      if (k < npages) hm[h] = fmaxf(hm[h], s);
      const long long row = ((long long)(b * a.Hq + h0 + h)) * a.cand_stride;
      if (k < npages) {
        if (j == 0) a.scores[row + slot] = s;
        if (DOTS) a.dots[(row + slot) * 4 + j] = valid ? I : 0;
      }
    }
   }
  }
  // ---- next chunk of this workgroup, if any (block-uniform)
  wg_first += gridDim.x * 4 * a.pw;
  if (wg_first >= count) break;
  first = wg_first + wave * a.pw;
  my_lp = -1; my_pool = -1;
  if (lane < a.pw && first + lane < count) {
    my_lp = FULL ? first + lane : a.sel_pages[((long long)(b * a.Hq + h0)) * a.max_sel + first + lane];
    if (my_lp >= 0 && my_lp < P) {
      const int pp = a.page_table[(long long)b * a.max_pages + my_lp];
      if (pp >= 0 && pp < a.pool_pages) my_pool = pp;
    }
  }
  npages = count - first;
  if (npages > a.pw) npages = a.pw;
  }
  if (a.headmax) {
    // one atomic per head and workgroup: waves reduce through LDS first
    __shared__ float hm_s[4][NH];
#pragma unroll
    for (int h = 0; h < NH; ++h) {
      const float mx = tw_wave_max_f(hm[h]);
      if (lane == 0) hm_s[wave][h] = mx;
    }
    __syncthreads();
    if (tid < NH) {
      const float mx = fmaxf(fmaxf(hm_s[0][tid], hm_s[1][tid]), fmaxf(hm_s[2][tid], hm_s[3][tid]));
      if (mx > -__builtin_inff())
        atomicMax(a.headmax + ((long long)(b * a.Hq + h0 + tid) * HM_SLOTS + (blockIdx.x & (HM_SLOTS - 1))) * TW_CTR, tw_float_key(mx));
    }
  }
}

// ------------------------------------------------------------------ int4_score over token lists
// The candidates of a head are token positions handed over by any token-level selector
// (Section 4.1).  A quad of lanes owns one candidate (lane & 3 = group of 32 dims): 16 bytes of
// codes and the group's (scale, zero) per lane, gathered from the token's slot in its page; a
// workgroup covers 256 consecutive candidate slots, 64 per step, all steps' loads in flight
// together.  Same integers and fp32 operations as the page-list kernel: bit-identical scores.
template <bool DOTS, int BITS>
__global__ __launch_bounds__(256) void int4_score_tokens_kernel(ScoreArgs a) {
  constexpr int IT = 4;
  const int tid = threadIdx.x, j = tid & 3;
  const int b = blockIdx.y / a.Hq, h0 = blockIdx.y % a.Hq, g = h0 / (a.Hq / a.Hkv);
  // (at least 0: the bound of the unsigned comparison below, and an empty sequence's length may be negative)
  const int ntok = max(0, min(a.seq_lens[b], a.max_pages * TW_PAGE));
  int count = a.sel_count[b * a.Hq + h0];
  if (count > a.max_sel) count = a.max_sel;
  // chunk columns as in the page-list kernel: a grid a multiple of 8 wide is rotated by the KV group's number
  const int col = a.rotate ? (int)((blockIdx.x + gridDim.x - ((unsigned)(b * a.Hkv + g) & 7u)) % gridDim.x) : (int)blockIdx.x;
  int wg_first = col * 64 * IT;
  if (a.arrive && blockIdx.x == 0 && tid == 0) a.arrive[(b * a.Hkv + g) * TW_CTR] = 0;
  if (wg_first >= count) return;

  // token -> pool slot of every step first, so that the dependent loads overlap the query prologue
  const long long row = ((long long)(b * a.Hq + h0)) * a.cand_stride;
  long long slot4[IT];                              // (token slot in the pool) * 4 + group, or -1
  auto translate = [&]() {
    // unconditional loads at clamped places (by minima: a selected index became a branch with a wait of its own), so
    // that no step's wait for another's: 33.6 -> 30.4 us for 256 heads x 4096 of 32768 tokens
    uint32_t tok[IT], pp[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int c = wg_first + it * 64 + (tid >> 2);
      tok[it] = a.sel_pages[row + min(c, count - 1)];
    }
#pragma unroll
    for (int it = 0; it < IT; ++it)
      pp[it] = a.page_table[(long long)b * a.max_pages + (min(tok[it], (uint32_t)max(ntok - 1, 0)) >> 4)];
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const bool ok = (tok[it] < (uint32_t)ntok) & (wg_first + it * 64 + (tid >> 2) < count) & ((long long)pp[it] < a.pool_pages);
      const long long slot = (((((long long)pp[it] * a.Hkv + g) * TW_PAGE + (tok[it] & 15)) << 2) + j);
      slot4[it] = ok ? slot : -1ll;
    }
  };
  translate();

  __shared__ int qi_s[1][32];
  __shared__ float c_s[1];
  tw_quantize_q<1>(a.q + ((long long)(b * a.Hq + h0)) * 128, qi_s, c_s);
  int qw[8], qs, i0;
  tw_query_words<BITS>(qi_s[0] + 8 * j, qw, &qs, &i0);
  const float qsf = (float)qs, cc = c_s[0];

#pragma unroll 1
  for (;;) {
    uint4 raw[IT][BITS == 8 ? 2 : 1];
    uint32_t meta[IT];
#pragma unroll
    for (int it = 0; it < IT; ++it) {               // unconditional loads (an invalid candidate reads slot 0, masked below)
      const long long idx = slot4[it] >= 0 ? slot4[it] : (long long)j;
      tw_load_raw<BITS>(a.kq_pool, idx, raw[it]);
      meta[it] = a.kq_meta[idx];
    }
#pragma unroll
    for (int it = 0; it < IT; ++it) {
      const int c = wg_first + it * 64 + (tid >> 2);
      const bool valid = slot4[it] >= 0;
      const int I = tw_group_dot<BITS>(qw, raw[it], i0);
      const float T = tw_token_sum(meta[it], I, qsf);   // all four lanes of the quad take part
      const float sc = valid ? __fmul_rn(T, cc) : -__builtin_inff();
      if (c < count) {
        if (j == 0) a.scores[row + c] = sc;
        if (DOTS) a.dots[(row + c) * 4 + j] = valid ? I : 0;
      }
    }
    wg_first += gridDim.x * 64 * IT;                // next chunk of this workgroup, if any (block-uniform)
    if (wg_first >= count) break;
    translate();
  }
}

// ------------------------------------------------------------------ int4_score on the matrix cores
// Every page a candidate and 4 or 8 query heads per KV head: per page the scores are a small dense
// contraction, [heads x 128 dims] . [128 dims x 16 tokens], which on the vector ALU costs 8 dot4
// per lane and head and 64 registers of query words (8 heads: 130 VGPRs, 3 waves per SIMD, too few
// pages in flight to keep HBM busy).  Here v_mfma_i32_16x16x32_i8 does the integer part.  The four
// groups of 32 dims have their own (scale, zero), so their dot products must stay apart: row
// 4*h + j of the A operand carries head h's query words of group j and zeros elsewhere, and lane
// (k-block j', token t) supplies group j' of token t as B; four MFMAs (one per 8-dim word of the
// groups) accumulate I_j[h][t].  The result lands with lane (h, t) holding I_0..I_3: scale/zero,
// the fixed-order sum and the store need no cross-lane step.  Same integers and the same fp32
// operations as the vector kernel, so the scores are bit-identical.
typedef int tw_i32x4 __attribute__((ext_vector_type(4)));

// HIST: the long-row pruner's histogram (topp_common.h) is made here, while the scores are in registers: one integer LDS
// add per score in a kernel that waits for memory.  At 4 x 64 heads x 262144 tokens it costs 9 us of 185, a pass over
// the stored scores 55 us.  (Floating-point LDS adds of the scores' weights: 360 us.)
template <int NHG, bool DOTS, int UNR, bool HIST = false>           // NHG groups of 4 heads
__global__ __launch_bounds__(256) void int4_score_mfma_kernel(ScoreArgs a) {
  constexpr int NH = 4 * NHG;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int b = blockIdx.y / a.Hkv, g = blockIdx.y % a.Hkv, h0 = g * NH;
  const int n = a.seq_lens[b];
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  const int count = P;
  const int wg_first = blockIdx.x * 4 * a.pw;
  if (a.arrive && blockIdx.x == 0 && tid == 0) a.arrive[(b * a.Hkv + g) * TW_CTR] = 0;
  if (wg_first >= count) return;

  // ---- this wave's pages: lane k holds the k-th one (logical id, pool id)
  const int first = wg_first + wave * a.pw;
  int my_lp = -1, my_pool = -1;
  if (lane < a.pw && first + lane < count) {
    my_lp = first + lane;
    const int pp = a.page_table[(long long)b * a.max_pages + my_lp];
    if (pp >= 0 && pp < a.pool_pages) my_pool = pp;
  }
  int npages = count - first;
  if (npages > a.pw) npages = a.pw;

  __shared__ int qi_s[NH][32];
  __shared__ float c_s[NH];
  __shared__ uint32_t hist_s[HIST ? NH * WH_LDS : 1];
  float hinv[NHG], hoff[NHG], hls[NHG];          // t = s * hinv + hoff
  if (HIST) {
    for (int i = tid; i < NH * WH_LDS; i += 256) hist_s[i] = 0;
#pragma unroll
    for (int hg = 0; hg < NHG; ++hg) {
      const WhGrid gr = a.hgrid[b * a.Hq + h0 + hg * 4 + (lane >> 4)];
      hinv[hg] = 1.0f / gr.scale;
      hoff[hg] = -gr.ref * hinv[hg];
      hls[hg] = gr.scale * kLog2e;
    }
  }
  tw_quantize_q<NH>(a.q + ((long long)(b * a.Hq + h0)) * 128, qi_s, c_s, a.chmask ? a.chmask + g * 4 : nullptr);

  const int kb = lane >> 4, t = lane & 15;       // B operand / result: k-block (= group of dims) or head, token
  // A operand: row m = lane & 15 = 4 * head + group; this lane's k-block only meets its own group
  long aw[NHG][4];
  {
    const int hl = t >> 2, j = t & 3;
#pragma unroll
    for (int hg = 0; hg < NHG; ++hg)
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        uint32_t lo = (uint32_t)qi_s[hg * 4 + hl][8 * j + 2 * w], hi = (uint32_t)qi_s[hg * 4 + hl][8 * j + 2 * w + 1];
        if (kb != j) { lo = 0; hi = 0; }
        aw[hg][w] = (long)(((unsigned long long)hi << 32) | lo);
      }
  }
  // result side: this lane's head is kb (+ 4 per head group); sums of its query words per group
  float qsf[NHG][4], cc[NHG];
#pragma unroll
  for (int hg = 0; hg < NHG; ++hg) {
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      int qs = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) qs = __builtin_amdgcn_sdot4(qi_s[hg * 4 + kb][8 * j + k], 0x01010101, qs, false);
      qsf[hg][j] = (float)qs;
    }
    cc[hg] = c_s[hg * 4 + kb];
  }

  float hm[NHG];
#pragma unroll
  for (int hg = 0; hg < NHG; ++hg) hm[hg] = -__builtin_inff();
#pragma unroll 1
  for (int k0 = 0; k0 < npages; k0 += UNR) {
    uint4 nib[UNR], mt[UNR];
    int lpv[UNR];
    bool okv[UNR];
#pragma unroll
    for (int kk = 0; kk < UNR; ++kk) {           // unconditional loads (an absent page reads pool page 0, masked below)
      const int k = k0 + kk;
      lpv[kk] = __builtin_amdgcn_readlane(my_lp, k & 63);
      const int pool = k < npages ? __builtin_amdgcn_readlane(my_pool, k & 63) : -1;
      okv[kk] = pool >= 0;
      const long long blk = ((long long)(pool >= 0 ? pool : 0) * a.Hkv + g) * 64;
      // every page is read once here (all heads of the group in this workgroup): non-temporal loads
      nib[kk] = tw_ld_stream(a.kq_pool + blk + t * 4 + kb);                // group kb of token t: 32 codes
      mt[kk] = tw_ld_stream((const uint4*)a.kq_meta + (blk >> 2) + t);     // token t: 4 x (scale | zero << 16)
    }
#pragma unroll
    for (int kk = 0; kk < UNR; ++kk) {
      const int k = k0 + kk;
      if (k < npages) {                          // wave-uniform
        const uint32_t wv[4] = {nib[kk].x, nib[kk].y, nib[kk].z, nib[kk].w};
        long bw[4];
#pragma unroll
        for (int w = 0; w < 4; ++w)
          bw[w] = (long)(((unsigned long long)((wv[w] >> 4) & 0x0F0F0F0Fu) << 32) | (wv[w] & 0x0F0F0F0Fu));
        const uint32_t mv[4] = {mt[kk].x, mt[kk].y, mt[kk].z, mt[kk].w};
        const int tok = lpv[kk] * TW_PAGE + t;
        const bool valid = okv[kk] && tok < n;
        const long long slot = (long long)(first + k) * TW_PAGE + t;
#pragma unroll
        for (int hg = 0; hg < NHG; ++hg) {
          tw_i32x4 c = {0, 0, 0, 0};
#pragma unroll
          for (int w = 0; w < 4; ++w) c = __builtin_amdgcn_mfma_i32_16x16x32_i8(aw[hg][w], bw[w], c, 0, 0, 0);
          float T[4];
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const float sc = __half2float(__ushort_as_half((unsigned short)(mv[j] & 0xFFFFu)));
            const float ze = __half2float(__ushort_as_half((unsigned short)(mv[j] >> 16)));
            T[j] = __fadd_rn(__fmul_rn(sc, (float)c[j]), __fmul_rn(ze, qsf[hg][j]));
          }
          const float ssum = __fadd_rn(__fadd_rn(T[0], T[1]), __fadd_rn(T[2], T[3]));
          const float s = valid ? __fmul_rn(ssum, cc[hg]) : -__builtin_inff();
          hm[hg] = fmaxf(hm[hg], s);
          const long long row = ((long long)(b * a.Hq + h0 + hg * 4 + kb)) * a.cand_stride;
          a.scores[row + slot] = s;
          if (HIST) {
            uint32_t w;
            const int bk = wh_bucket(__builtin_fmaf(valid ? s : 0.f, hinv[hg], hoff[hg]), hls[hg], &w);
            atomicAdd(&hist_s[(hg * 4 + kb) * WH_LDS + bk], valid ? w : 0u);
          }
          if (DOTS) ((tw_i32x4*)a.dots)[row + slot] = valid ? c : tw_i32x4{0, 0, 0, 0};
        }
      }
    }
  }
  if (a.headmax) {
    // one atomic per head and workgroup: 16-lane rows (one head each), then the waves through LDS
    __shared__ float hm_s[4][NH];
#pragma unroll
    for (int hg = 0; hg < NHG; ++hg) {
      float mx = hm[hg];
      mx = fmaxf(mx, tw_dpp_f<TW_DPP_XOR1>(mx));
      mx = fmaxf(mx, tw_dpp_f<TW_DPP_XOR2>(mx));
      mx = fmaxf(mx, tw_dpp_f<TW_DPP_HALF_MIRROR>(mx));
      mx = fmaxf(mx, tw_dpp_f<TW_DPP_MIRROR>(mx));
      if (t == 0) hm_s[wave][hg * 4 + kb] = mx;
    }
    __syncthreads();
    if (tid < NH) {
      const float mx = fmaxf(fmaxf(hm_s[0][tid], hm_s[1][tid]), fmaxf(hm_s[2][tid], hm_s[3][tid]));
      if (mx > -__builtin_inff())
        atomicMax(a.headmax + ((long long)(b * a.Hq + h0 + tid) * HM_SLOTS + (blockIdx.x & (HM_SLOTS - 1))) * TW_CTR, tw_float_key(mx));
    }
  }
  if (HIST) {
    __syncthreads();
    for (int i = tid; i < NH * WH_NB; i += 256) {
      const int h = i / WH_NB, k = i % WH_NB;
      const uint32_t c = hist_s[h * WH_LDS + k];
      if (c) atomicAdd(a.ghist + (long long)(b * a.Hq + h0 + h) * WH_NB + k, (unsigned long long)c);
    }
  }
}

// ------------------------------------------------------------------ sample of a row, for its histogram's grid
// Ahead of the full-row scoring of the long-row pruner: one workgroup per query head scores 64 pages spread evenly over
// the sequence (8 waves x 8 pages), and the top-p threshold of the sampled scores (to 1/256 of their range) and their
// weighted deviation place the head's histogram.  The workgroups beyond the heads clear the workspace words that the passes behind this one add to.
// Bound by its chain of dependent loads; one workgroup per KV head, scoring its heads one after the other on
// batch * Hkv of the 256 CUs, took 18.8 us at 4 x 8 groups of 8 heads, this 10.4.
struct SampleArgs {
  ScoreArgs s;
  WhGrid* hgrid;
  uint4* zero;
  long long zero16;
  int heads;                  // batch * Hq
  float p;
};
constexpr int SMP_NT = 512, SMP_ZERO_WGS = 256;

__global__ __launch_bounds__(SMP_NT) void row_sample_kernel(SampleArgs sa) {
  constexpr int NW = SMP_NT / 64, K = 64 / NW;
  const ScoreArgs& a = sa.s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if ((int)blockIdx.x >= sa.heads) {
    for (long long i = (long long)(blockIdx.x - sa.heads) * SMP_NT + tid; i < sa.zero16; i += (long long)SMP_ZERO_WGS * SMP_NT)
      sa.zero[i] = make_uint4(0, 0, 0, 0);
    return;
  }
  const int bh = blockIdx.x, b = bh / a.Hq, h = bh % a.Hq, g = h / (a.Hq / a.Hkv);
  const int n = a.seq_lens[b];
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  uint4 raw[K][1];
  uint32_t meta[K];
  int lp[K];
  bool ok[K];
#pragma unroll
  for (int k = 0; k < K; ++k) {
    lp[k] = (int)(((long long)(wave * K + k) * P) >> 6);           // below P (0 when there is none)
    const int pp = a.page_table[(long long)b * a.max_pages + lp[k]];
    ok[k] = P > 0 && pp >= 0 && pp < a.pool_pages;
    const long long blk = ((long long)(ok[k] ? pp : 0) * a.Hkv + g) * 64;
    tw_load_raw<4>(a.kq_pool, blk + lane, raw[k]);
    meta[k] = a.kq_meta[blk + lane];
  }
  __shared__ int qi_s[1][32];
  __shared__ float c_s[1];
  __shared__ float mx_s[NW], sum_s[NW][3];
  tw_quantize_q<1, SMP_NT>(a.q + (long long)bh * 128, qi_s, c_s);
  const int j = lane & 3;
  int qw[8], qs, i0;
  tw_query_words<4>(qi_s[0] + 8 * j, qw, &qs, &i0);
  float sv[K], mx = -__builtin_inff();
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float T = tw_token_sum(meta[k], tw_group_dot<4>(qw, raw[k], i0), (float)qs);
    sv[k] = ok[k] && lp[k] * TW_PAGE + (lane >> 2) < n ? __fmul_rn(T, c_s[0]) : -__builtin_inff();
    mx = fmaxf(mx, sv[k]);
  }
  mx = tw_wave_max_f(mx);
  if (lane == 0) mx_s[wave] = mx;
  __syncthreads();
  mx = mx_s[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) mx = fmaxf(mx, mx_s[w]);
  const bool some = mx > -__builtin_inff() && mx < __builtin_inff();
  float w0 = 0.f, w1 = 0.f, w2 = 0.f;              // (all four lanes of a token's quad: the sums' ratios do not mind)
#pragma unroll
  for (int k = 0; k < K; ++k) {
    if (some && sv[k] > -__builtin_inff()) {
      const float t = sv[k] - mx, w = __expf(t);
      w0 += w; w1 += w * t; w2 += w * t * t;
    }
  }
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) { w0 += __shfl_xor(w0, o, 64); w1 += __shfl_xor(w1, o, 64); w2 += __shfl_xor(w2, o, 64); }
  if (lane == 0) { sum_s[wave][0] = w0; sum_s[wave][1] = w1; sum_s[wave][2] = w2; }
  __syncthreads();
  __shared__ uint32_t hist_s[256];
  if (tid < 256) hist_s[tid] = 0;
  __syncthreads();
  w0 = w1 = w2 = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) { w0 += sum_s[w][0]; w1 += sum_s[w][1]; w2 += sum_s[w][2]; }
  WhGrid gr = wh_grid(w0, w1, w2);                 // ref relative to mx, and below it
  const float reach = 16.0f * gr.scale - gr.ref;   // from the maximum to four deviations below that first guess
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const float d = mx - sv[k];
    if (some && j == 0 && d < reach) atomicAdd(&hist_s[(int)(d / reach * 255.0f)], (uint32_t)(__expf(-d) * 1048576.0f));
  }
  __syncthreads();
  if (wave == 0) {
    uint32_t c[4], mine = 0;
#pragma unroll
    for (int k = 0; k < 4; ++k) { mine += hist_s[4 * lane + k]; c[k] = mine; }
    const uint32_t incl = tw_wave_scan_u32(mine);
    const float target = sa.p * (float)__shfl(incl, 63, 64);
    int bin = 4 * lane + 3;
#pragma unroll
    for (int k = 2; k >= 0; --k) bin = (float)(incl - mine + c[k]) >= target ? 4 * lane + k : bin;
    const int at = __ffsll((long long)__ballot((float)incl >= target)) - 1;
    if (some && at >= 0) gr.ref = -((float)__shfl(bin, at, 64) + 0.5f) * (1.0f / 255.0f) * reach;
    if (some) gr.ref += mx;
    if (lane == 0) sa.hgrid[bh] = gr;
  }
}

// ------------------------------------------------------------------ top-p per head, scores in registers
// One workgroup of 256 to 1024 threads (the rules at launch_topp) per
// (sequence, query head); thread t owns the contiguous candidate slots
// [t*EPT, (t+1)*EPT).  Rank (fixed-point distance to the max logit) and softmax
// numerator of every score are computed once and stay in registers, or are
// recomputed where those are short.  Pass 0
// buckets the ranks within 8 logits of the max at 1/64 logit and only sums up
// everything further down (no atomics); the crossing bucket is narrowed 9 bits
// per pass until at most HP_CAP scores remain, which are resolved exactly on the
// score's own bits.  Every wave scans the histogram on its own, so a pass costs
// one barrier.  The kept tokens are written as a bitmap over token positions;
// the last head of a KV group to arrive turns the group's bitmaps into the
// sorted union.
struct HeadArgs {
  const float* scores;
  float* scores_w;            // FUSE == 3: the same rows, written here
  const int32_t* sel_pages;
  const int32_t* sel_count;
  const int32_t* seq_lens;
  int32_t* kept_count;
  int32_t* kept_idx;          // or nullptr
  uint32_t* bitmaps;          // [b][Hq][words_stride]
  uint32_t* arrive;           // [b][Hkv] arrival counters, zero on entry
  int32_t* union_count;
  int32_t* union_idx;
  uint32_t* status;
  int Hq, Hkv, max_pages, max_sel, cand_stride, kept_stride, words_stride, union_stride;
  int n_above, n_upto;        // this launch takes the heads with n_above < candidates <= n_upto
  float p;
  // scoring inside the kernel (FUSE): the query, the quantised copy of K and the page table
  const uint16_t* q;
  const int32_t* page_table;
  const uint4* kq_pool;
  const uint32_t* kq_meta;
  long long pool_pages;
  int remap;                  // FUSE: workgroup -> head mapping that keeps the heads of a KV head on one XCD
  // page selection inside the kernel as well (FUSE == 2): the bounds of all pages and the budgets; the lists go
  // to sel_pages_w / sel_count_w
  const float* bounds;        // [b][Hq][max_pages]
  const int32_t* budget;      // [b] tokens
  int32_t* sel_pages_w;
  int32_t* sel_count_w;
  int parts;                  // FUSE == 3: workgroups per head
  int ordered;                // FUSE == 2, 4: sequences are taken in the order that the kernel before left (tw_order_word)
};

constexpr int HP_CAP = 64;                    // exact resolve handles up to this many scores
constexpr int HP_BITMAP_WORDS = 6144;         // 196608 tokens
constexpr int HP_USTAGE = 4096;               // union lists up to this length leave through LDS

// TOK: the candidates are token positions (sel_pages = the token lists, max_sel = their row length,
// sel_count in tokens) instead of pages of 16 slots.
// FUSE >= 1: the estimated scores are computed here, from the head's page list, instead of being read from the row a
// scoring launch wrote: the workgroup's waves share the list (one page of 64 (token, group) lanes per wave and step,
// the arithmetic of int4_score_kernel), the scores cross to their owner threads through LDS.
// FUSE == 2: the page list too is made here, from the bounds of all pages (the selection of page_select_reg_kernel).
// FUSE == 3: the same with a.parts workgroups per head, for few heads with long lists, whose lists one workgroup per head
// pulls too slowly.  Each selects the head's pages (the same list in each), scores its share of them into the head's row,
// and the last one to get there goes on with top-p alone (1 x 32 heads x 8192 pages, 8192 candidates: page_select 6.6 +
// int4_score 5.0 + topp 19.2 us -> 30.4; 4 x 32 heads x 4096 pages 35.5 -> 32.0).
// FUSE == 4: FUSE == 2 with the scores in registers where that would leave them in LDS.
// BITS: width of the quantised copy's codes (FUSE >= 2; else 4).
template <int NT, int EPT, int G, bool TOK = false, int FUSE = 0, int BITS = 4>
__global__ __launch_bounds__(NT, NT > 512 ? 1 : (FUSE == 2 && EPT == 8 ? 8 : (FUSE != 2 && EPT > 8 ? 4 : 6))) void topp_head_kernel(HeadArgs a) {
  constexpr int NW = NT / 64;
  constexpr bool SELECT = FUSE >= 2, SPLIT = FUSE == 3;
  // The workgroups that are there to share a CU (many heads, 8 or 16 candidates per thread, scored here) leave the scores
  // in LDS, where every phase reads them again, instead of holding them in registers: three of 16 candidates per thread
  // fit a CU instead of two, four of 8 instead of three, and one's scoring streams while the others wait at barriers
  // (64 ragged sequences x 32 heads 116.6 -> 104.0 us, 32 x 32 heads x 4096 candidates 56.2 -> 53.7).  The price is in the phases:
  // reading the scores again, 64 registers (74 with 16 candidates per thread) of which the form with 8 spills 8, 36 bytes of
  // scratch per lane.  Where four to a CU do not save a round of workgroups over three, FUSE == 4 is quicker (launch_topp).
  constexpr bool INLDS = FUSE == 2 && NT <= 512 && EPT > 4;
  // Arguments of the last phases read again there, where keeping them takes more scalar registers than there are: 6 to 40 of them went
  // back and forth between scalar and vector ones all the way (21 of the form with four to a CU still do).  Each is a trip to the scalar
  // cache behind the search's barriers, which the other forms lose by: token lists of 256 heads 8.0 us, 7.55 without, of 32 7.6 / 7.3,
  // page lists of 32 heads 10.8 / 10.6.
  constexpr bool LATE = INLDS || SPLIT || FUSE == 4 || (FUSE == 1 && EPT == 16);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const unsigned parts = SPLIT ? (unsigned)a.parts : 1u;
  int b_ = blockIdx.y, h_ = blockIdx.x / parts, part = blockIdx.x % parts;
  if (FUSE && a.remap) {
    // Workgroups go to the 8 XCDs round robin in dispatch order.  The G heads of a KV head select largely the
    // same pages: they take G consecutive workgroups of one XCD, so that each finds the others' pages in its L2.
    const unsigned L = blockIdx.y * gridDim.x + blockIdx.x, xcd = L & 7u, r = L >> 3;
    const unsigned grp = (r / (G * parts)) * 8u + xcd;   // (sequence, KV head), batch * Hkv a multiple of 8
    b_ = (int)(grp / (unsigned)a.Hkv);
    h_ = (int)(grp % (unsigned)a.Hkv) * G + (int)(r / parts % G);
    part = (int)(r % parts);
  }
  // (the most work first: 64 ragged sequences x 32 heads 95.5 -> 79 us, 40 x 32 72.6 -> 55, 16 x 64 42.5 -> 35)
  if ((FUSE == 2 || FUSE == 4) && a.ordered) b_ = __builtin_amdgcn_readfirstlane((int)a.arrive[tw_order_word(b_, a.Hkv)]);
  const int b = b_, h = h_;
  const int bh = b * a.Hq + h;
  // SELECT: everything the page selection reads is asked for here, before the sequence's length is known (any
  // entry of the head's row of bounds and of the sequence's page-table row may be read): the bounds and the
  // page-table entries of the pages j * NT + tid, which this thread will list (1024-thread workgroups, 4 entries each;
  // the smaller ones, short of registers, ask when they know the length)
  // SELECT with few candidates: the row of pages is bounded too (the launch's rule), and LDS is sized for that
  constexpr bool SMALL = FUSE == 2 && NT <= 512 && EPT == 4;
  constexpr int SEL_E = SMALL ? 4 : (SPLIT ? 8192 : 4096) / NT;
  constexpr int BWORDS = SELECT ? SEL_E * NT * TW_PAGE / 32 : HP_BITMAP_WORDS;
  constexpr int USTAGE = SMALL ? 4 * NT : HP_USTAGE;
  constexpr int AREA = SELECT ? (NT * EPT > USTAGE ? NT * EPT : USTAGE) : USTAGE;
  constexpr bool SEL_EARLY = SELECT && NT >= 1024;
  const int n = a.seq_lens[b];
  const int budget_b = SELECT ? a.budget[b] : 0;
  float sel_pre[SELECT ? SEL_E : 1];
  int32_t sel_pt[SELECT ? SEL_E : 1];
  auto ask_selection = [&]() {
#pragma unroll
    for (int j = 0; j < SEL_E; ++j) {
      const int i = j * NT + tid < a.max_pages ? j * NT + tid : a.max_pages - 1;
      sel_pre[SEL_EARLY ? j : 0] = a.bounds[(long long)bh * a.max_pages + i];
      sel_pt[SEL_EARLY ? j : 0] = a.page_table[(long long)b * a.max_pages + i];
    }
  };
  // FUSE: this lane's pair of the query's elements, asked for early too (bf16 rows may begin at any element: no more than 2-byte alignment)
  uint32_t q_raw = 0u;
  if (FUSE) {
    if (SEL_EARLY) ask_selection();
    __builtin_memcpy(&q_raw, a.q + (long long)bh * 128 + 2 * lane, 4);
    __builtin_amdgcn_sched_barrier(0);               // these loads are issued before anything below waits for the lengths
  }
  int P = n > 0 ? (n + TW_PAGE - 1) / TW_PAGE : 0;
  if (P > a.max_pages) P = a.max_pages;
  const int ntok = P * TW_PAGE < n ? P * TW_PAGE : n;
  const int nwords = (ntok + 31) >> 5;
  int count;
  if (SELECT) {
    int P2;
    tw_select_sizes<TW_PAGE>(n, budget_b, a.max_pages, a.max_sel, &P2, &count);
  } else {
    count = a.sel_count[bh];
    if (count > a.max_sel) count = a.max_sel;
    if (count < 0) count = 0;
  }
  const int N = TOK ? count : count * TW_PAGE;
  if (N <= a.n_above || N > a.n_upto) return;     // another launch's head (block-uniform)
  const float* row = a.scores + (long long)bh * a.cand_stride;
  const int c0 = tid * EPT;
  TW_STAMP(0);

  __shared__ unsigned long long histM[HP_NB];
  __shared__ uint32_t histC[HP_NB];
  __shared__ unsigned long long cand_mass[HP_CAP];
  __shared__ uint32_t cand_key[HP_CAP];
  // position bitmap, then the union list on its way out; before that the selection's arrays and the scores, read 16
  // bytes at a time: behind the bitmap (SELECT, whose bitmap covers the pages that its keys can be: NT * SEL_E) or from its first word
  __shared__ __align__(16) uint32_t big_s[BWORDS + AREA];
  static_assert(__alignof__(big_s) >= 16 && BWORDS % 4 == 0, "read as float4 and as 64-bit words");
  uint32_t* const bitmap = big_s;
  uint32_t* const area = SELECT ? big_s + BWORDS : big_s;
  int32_t* const ustage = (int32_t*)(big_s + BWORDS);
  __shared__ unsigned long long tail_s[NW];
  __shared__ uint32_t ws32[16];
  __shared__ float redf[NW];
  __shared__ uint32_t sh_n, sh_kept, sh_T, sh_last;

  __shared__ int32_t pages_s[SELECT ? NT * EPT / TW_PAGE : 1];   // SELECT: the head's page list ...
  __shared__ int32_t pool_s[SELECT ? NT * EPT / TW_PAGE : 1];    // ... and the pages' places in the pool
  if (SELECT) {
    // (SPLIT: up to 8192 bounds, most of them close together below a few large ones; with 512 buckets their adds queue on
    //  few words - 4.7 us of histogram, with 1024 2.1, with 2048 the scan takes what the adds save)
    constexpr int SNB = SPLIT ? 1024 : 512;
    static_assert(SNB % 2 == 0, "the candidates behind the histogram are 64-bit words");
    uint32_t* const hist = area;                    // the selection's arrays lie there
    unsigned long long* const cand = (unsigned long long*)(area + tw_sel_words(SNB));
    uint32_t* const cnt = area + tw_sel_words(SNB) + 2 * SEL_CAP;
    static_assert(tw_sel_words(SNB) + 2 * SEL_CAP + SEL_E * NT / 64 <= AREA, "the selection's arrays fit");
    int32_t* const out = a.sel_pages_w + (long long)bh * a.max_sel;
    const int32_t* const ptab = a.page_table + (long long)b * a.max_pages;
    if (tid == 0 && part == 0) a.sel_count_w[bh] = count;
    if (count == P) {                               // the budget covers the sequence (block-uniform)
      for (int i = tid; i < P; i += NT) { if (part == 0) out[i] = i; pages_s[i] = i; pool_s[i] = ptab[i]; }
    } else if (count > 0) {
      if (!SEL_EARLY) {
        const float* const sc = a.bounds + (long long)bh * a.max_pages;
#pragma unroll
        for (int e = 0; e < SEL_E; ++e) {
          if (e * NT >= P) continue;                 // (block-uniform)
          const int i = e * NT + tid < P ? e * NT + tid : P - 1;
          sel_pre[SELECT ? e : 0] = sc[i];
          sel_pt[SELECT ? e : 0] = ptab[i];
        }
      }
      uint32_t key[SEL_E], T, need_eq;
#pragma unroll
      for (int e = 0; e < SEL_E; ++e) key[e] = tw_float_key(sel_pre[SELECT ? e : 0]);
      tw_select_threshold<NT, SEL_E, SNB, 30>(key, P, (uint32_t)count, hist, cand, &T, &need_eq);
      tw_select_list<NT, SEL_E>(key, P, T, need_eq, cnt, [&](uint32_t pos, int e) {
        if (pos < (uint32_t)a.max_sel) {
          if (part == 0) out[pos] = e * NT + tid;
          pages_s[pos] = e * NT + tid;
          pool_s[pos] = sel_pt[SELECT ? e : 0];
        }
      });
    }
    __syncthreads();                                // list complete; the area free for the scores
    TW_STAMP(35);
  }

  // ---- scores into registers; logical pages of the owned slots
  // (loads do not wait for the list length: anything inside the row is readable, slots at or
  //  beyond N are masked afterwards)
  constexpr int NPG = TOK ? EPT : INLDS ? EPT / 4 : (EPT + 15) / 16; // pages a thread's slots fall into (a part of one if EPT < 16); TOK: one token per slot
  constexpr int SN = INLDS ? 1 : EPT;
  float s[SN];
  int pg[NPG];
  float* const sc_s = (float*)area;
  if (FUSE) {
    static_assert(NT * EPT <= (SELECT ? AREA : BWORDS + USTAGE), "scores of a row must fit the staging array");
    __shared__ __align__(16) int qi_s[NW][32];
    // this wave's share of the list: lane k holds its k-th page
    static_assert(EPT * 64 / TW_PAGE <= 64, "a wave's share of the longest list has a lane for every page");
    constexpr int UF = (!SPLIT && NT >= 1024 || EPT == 4 || (INLDS && EPT == 16) ? 8 : 4) / (BITS == 8 ? 2 : 1);   // pages in flight per wave (register budget)
    // SPLIT: this workgroup's share of the list
    const int share = SPLIT ? (count + (int)parts - 1) / (int)parts : count, share0 = SPLIT ? part * share : 0;
    const int share1 = share0 + share < count ? share0 + share : count;
    const int ppw = INLDS || SPLIT ? (share + NW - 1) / NW : ((share + NW - 1) / NW + UF - 1) / UF * UF;
    const int first = share0 + __builtin_amdgcn_readfirstlane(wave) * ppw;   // (scalar: the loop below is wave-uniform)
    int my_lp = -1, my_pool = -1;
    if (lane < ppw && first + lane < share1) {
      my_lp = SELECT ? pages_s[first + lane] : a.sel_pages[(long long)bh * a.max_sel + first + lane];
      if (my_lp >= 0 && my_lp < P) {
        const int pp = SELECT ? pool_s[first + lane] : a.page_table[(long long)b * a.max_pages + my_lp];
        if (pp >= 0 && pp < a.pool_pages) my_pool = pp;
      }
    }
    int npages = share1 - first;
    npages = npages < 0 ? 0 : (npages > ppw ? ppw : npages);
    const int j = lane & 3, g = h / G;
    int qw[8], i0;
    float qsf, cc;
    // UF pages in flight per wave.  Several workgroups to a CU: as a ring - a page's codes and (scale, zero) words are asked
    // for in the registers of the page used last, so that loads keep going out while the wave computes (unconditional, or
    // the wait for one page would take in the pages behind it: one past the wave's last reads as zeros); 2 us of the two
    // times above.  One workgroup to a CU, whose waves have a round or two each: in rounds, all of
    // a round's loads first (8 x 32 heads x 256 pages 22.0 us, as a ring 23.9).  Lanes past the wave's last page hold pool
    // -1; what the rounds store for them lies beyond the list (inside the array: NW * ppw <= NT * EPT / 16 pages).
    uint4 nib[UF][BITS == 8 ? 2 : 1];
    uint32_t meta[UF];
    auto ask = [&](int kk, int k) {
      const int pl = INLDS && k >= npages ? -1 : __builtin_amdgcn_readlane(my_pool, k & 63);   // (lanes past the last page hold -1)
      tw_load_page<BITS>(a.kq_pool, a.kq_meta, (long long)pl * a.Hkv + g, pl >= 0, lane, nib[kk], &meta[kk]);
    };
    // every lane of a quad stores the token's score (same word)
    auto put = [&](int k, float sc) {
      const int slot = (first + k) * TW_PAGE + (lane >> 2);
      if (!SPLIT) sc_s[slot] = sc;
      else if (k < npages) __hip_atomic_store(a.scores_w + (long long)bh * a.cand_stride + slot, sc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    };
    auto use = [&](int kk, int k) { put(k, __fmul_rn(tw_token_sum<true>(meta[kk], tw_group_dot<BITS>(qw, nib[kk], i0), qsf), cc)); };
    // The first pages are asked for, then the query is quantised, by every wave on its own (by two of them for all, two barriers ahead of
    // the first load: 48 ragged sequences x 32 heads 36.1 -> 35.1 us, 4 x 32 heads of 8-bit codes 14.9 -> 14.4, the step of 1 x 4096 tokens 21.8 -> 21.6).
#pragma unroll
    for (int kk = 0; kk < UF; ++kk) ask(kk, kk);
    __builtin_amdgcn_sched_barrier(0);
    {
      int qs;
      int* const qi = qi_s[__builtin_amdgcn_readfirstlane(wave)];
      cc = tw_quantize_q1(q_raw, qi);
      tw_query_words<BITS>(qi + 8 * j, qw, &qs, &i0);
      qsf = (float)qs;
    }
    int k0 = 0;
    if (INLDS) {
#pragma unroll 1
      for (; k0 + UF < npages; k0 += UF) {
#pragma unroll
        for (int kk = 0; kk < UF; ++kk) {
          use(kk, k0 + kk);
          __builtin_amdgcn_sched_barrier(0);
          ask(kk, k0 + UF + kk);
          __builtin_amdgcn_sched_barrier(0);
        }
      }
#pragma unroll
      for (int kk = 0; kk < UF; ++kk)
        if (k0 + kk < npages) use(kk, k0 + kk);
    } else if (npages > 0) {
#pragma unroll 1
      for (;;) {
#pragma unroll
        for (int kk = 0; kk < UF; ++kk) use(kk, k0 + kk);
        k0 += UF;
        if (k0 >= npages) break;
#pragma unroll
        for (int kk = 0; kk < UF; ++kk) ask(kk, k0 + kk);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    // Pages that are not there, and the sequence's last one where it is not full: what does not count is stored anew.
    const int my_end = my_pool >= 0 ? n - my_lp * TW_PAGE : 0;      // tokens of this lane's page
    for (unsigned long long part_pages = __ballot(my_end < TW_PAGE && lane < npages); part_pages; part_pages &= part_pages - 1) {
      const int k = __ffsll((long long)part_pages) - 1;
      if ((lane >> 2) >= __builtin_amdgcn_readlane(my_end, k)) put(k, -__builtin_inff());
    }
    if (SPLIT) {
      // the hand-off of the bitmaps below: write-through stores, acknowledged, then one count per workgroup; the last one
      // reads the others' scores past the caches that are not shared by all compute units
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      __syncthreads();
      if (tid == 0)
        sh_last = __hip_atomic_fetch_add(a.arrive + (b * a.Hkv + h / G) * TW_CTR + 1 + h % G, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == parts - 1u ? 1u : 0u;
      __syncthreads();
      if (!sh_last) return;
      float x[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e) {
        const int i = e * NT + tid < a.cand_stride ? e * NT + tid : a.cand_stride - 1;
        x[e] = __hip_atomic_load(row + i, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int e = 0; e < EPT; ++e) sc_s[e * NT + tid] = x[e];
    }
    __syncthreads();
    if (!INLDS) {
#pragma unroll
      for (int v = 0; v < EPT / 4; ++v) {
        const float4 x = *(const float4*)(sc_s + c0 + 4 * v);
        s[(4 * v) % SN] = x.x; s[(4 * v + 1) % SN] = x.y; s[(4 * v + 2) % SN] = x.z; s[(4 * v + 3) % SN] = x.w;
      }
      if (FUSE == 1) __syncthreads();              // the bitmap, cleared below, lies in the same words
    }
  } else
#pragma unroll
  for (int v = 0; v < EPT / 4; ++v) {              // clamped, unconditional: all loads go out together
    const int cc = c0 + 4 * v < a.cand_stride ? c0 + 4 * v : a.cand_stride - 4;
    const float4 x = *(const float4*)(row + cc);
    s[(4 * v) % SN] = x.x; s[(4 * v + 1) % SN] = x.y; s[(4 * v + 2) % SN] = x.z; s[(4 * v + 3) % SN] = x.w;
  }
  if (TOK) {
#pragma unroll
    for (int v = 0; v < EPT / 4; ++v) {
      const int cc = c0 + 4 * v < a.max_sel ? c0 + 4 * v : a.max_sel - 4;
      const int4 x = *(const int4*)(a.sel_pages + (long long)bh * a.max_sel + cc);
      pg[(4 * v) % NPG] = x.x; pg[(4 * v + 1) % NPG] = x.y; pg[(4 * v + 2) % NPG] = x.z; pg[(4 * v + 3) % NPG] = x.w;
    }
  } else {
#pragma unroll
    for (int v = 0; v < NPG; ++v) {
      const int p0 = INLDS ? (v * 4 * NT + tid * 4) >> 4 : (c0 >> 4) + v, pi = p0 < a.max_sel ? p0 : a.max_sel - 1;
      pg[v] = SELECT ? pages_s[pi] : a.sel_pages[(long long)bh * a.max_sel + pi];
    }
  }
  if (!INLDS) {
#pragma unroll
    for (int e = 0; e < EPT; ++e) s[e % SN] = (c0 + e < N) ? s[e % SN] : -__builtin_inff();
  }
  // f(e, score) for this thread's slots
  auto each = [&](auto f) {
    if constexpr (INLDS) {
#pragma unroll
      for (int v = 0; v < EPT / 4; ++v) {
        if (EPT > 8 && v * 4 * NT >= N) break;     // (block-uniform; of 16 slots a thread most heads of a ragged batch fill few)
        const int at = v * 4 * NT + tid * 4;
        const float4 x = *(const float4*)(sc_s + at);
        f(4 * v, at < N ? x.x : -__builtin_inff());
        f(4 * v + 1, at + 1 < N ? x.y : -__builtin_inff());
        f(4 * v + 2, at + 2 < N ? x.z : -__builtin_inff());
        f(4 * v + 3, at + 3 < N ? x.w : -__builtin_inff());
      }
    } else {
#pragma unroll
      for (int e = 0; e < EPT; ++e) f(e, s[e % SN]);
    }
  };
  for (int i = tid; i < HP_NB; i += NT) { histM[i] = 0; histC[i] = 0; }
  for (int i = tid; i < nwords; i += NT) bitmap[i] = 0;
  if (tid == 0) { sh_n = 0; sh_kept = 0; }

  float m = -__builtin_inff();
  each([&](int, float x) { m = fmaxf(m, x); });
  m = tw_wave_max_f(m);
  if (lane == 0) redf[wave] = m;
  __syncthreads();
  m = redf[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) m = fmaxf(m, redf[w]);
  TW_STAMP(1);

  uint32_t T = 0;
  bool searching;
  if (!(m > -__builtin_inff())) { T = 0xFFFFFFFFu; searching = false; }
  else if (a.p >= 1.0f) { T = kKeyNegInf + 1u; searching = false; }
  else searching = true;

  if (searching) {                                 // block-uniform
    // rank and numerator of every score: computed once and kept, or (512-thread workgroups, which are there
    // to fit more of them on a CU) recomputed from the score where needed - a few instructions that save
    // 2 * EPT registers
    constexpr bool RECOMP = NT <= 512 && EPT > 4;
    uint32_t rk[RECOMP ? 1 : EPT];
    float ef[RECOMP ? 1 : EPT];
    if (!RECOMP) each([&](int e, float x) { rk[RECOMP ? 0 : e] = hp_rank(m, x, &ef[RECOMP ? 0 : e]); });
    auto rank_of = [&](int e, float x) -> uint32_t { return RECOMP ? hp_rank_only(m, x) : rk[RECOMP ? 0 : e]; };
    auto numer_of = [&](int e, float x) -> float { return RECOMP ? hp_numer(m, x) : ef[RECOMP ? 0 : e]; };
    uint32_t rlo = 0, pop = 0;
    int shift = 16, pass = 0;
    unsigned long long A = 0, target = 0;
#pragma unroll 1
    for (;;) {
      if (pass > 0) {
        for (int i = tid; i < HP_NB; i += NT) { histM[i] = 0; histC[i] = 0; }
        __syncthreads();
      }
      unsigned long long below = 0;                // mass past the end of the interval (pass 0 only)
      each([&](int e, float x) {
        const uint32_t r = rank_of(e, x);
        if (r != HP_NONE && r >= rlo) {
          const uint32_t bk = (r - rlo) >> shift;
          const unsigned long long w = hp_fix(numer_of(e, x));
          if (bk < HP_NB) { atomicAdd(&histM[bk], w); atomicAdd(&histC[bk], 1u); }
          else below += w;
        }
      });
      if (pass == 0) {
        below = tw_wave_scan_u64(below);
        if (lane == 63) tail_s[wave] = below;
      }
      __syncthreads();
      TW_STAMP(2 + pass);
      // every wave scans the 512 buckets on its own: lane l sums buckets 8l .. 8l+7; of the lane that holds the crossing
      // the first 8 lanes then take a bucket each: walking that lane's 8 sums in every wave took more vector instructions, which the
      // waves share their units for (step of 64 ragged sequences 230.0 -> 228.3 us), and registers for the sums where scores are held
      // in registers (1024 threads x 4 candidates 86 -> 64, x 8 102 -> 68, in parts 103 -> 80; the forms with scores in LDS: none)
      unsigned long long mine = 0;
#pragma unroll
      for (int k = 0; k < 8; ++k) mine += histM[8 * lane + k];
      const unsigned long long incl = tw_wave_scan_u64(mine);
      const unsigned long long total = tw_readlane_u64(incl, 63);
      if (pass == 0) {
        unsigned long long Z = total;
#pragma unroll
        for (int w = 0; w < NW; ++w) Z += tail_s[w];
        const double t = ceil((double)a.p * (double)Z);
        target = t < 1.0 ? 1ull : (unsigned long long)t;
        if (target > Z) target = Z;
      }
      const unsigned long long before = A + incl - mine;
      const bool hit = before < target && before + mine >= target;
      const unsigned long long bal = __ballot(hit);
      bool more = false;
      if (bal == 0 && pass == 0) {
        // not enough mass in the fine range: go on with everything below it
        A += total;
        rlo = HP_FINE_END; shift = 18;
        more = true;
      } else if (bal == 0) {
        pop = 0xFFFFFFFFu;                          // unreachable: the interval holds the crossing by construction
      } else {
        const int src = __ffsll((long long)bal) - 1;
        const unsigned long long c = histM[8 * src + (lane & 7)];
        const unsigned long long upto = tw_readlane_u64(before, src) + tw_scan8_u64(c);
        const int at = __ffsll((long long)__ballot(lane < 8 && upto >= target)) - 1;
        const int bucket = 8 * src + at;
        A = tw_readlane_u64(upto - c, at);
        pop = histC[bucket];
        rlo += (uint32_t)bucket << shift;
        if (pop > HP_CAP && shift > 0) { shift = shift >= 9 ? shift - 9 : 0; more = true; }
      }
      ++pass;
      if (!more) break;                             // same decision in every wave
      __syncthreads();                              // all scans done before the histogram is cleared
    }
    // the threshold lies among the `pop` scores with rank in [rlo, rlo + (1 << shift))
    const uint32_t rhi = rlo + (1u << shift) - 1u;
    const bool small = pop <= HP_CAP;
    uint32_t kmin = 0xFFFFFFFFu;
    each([&](int e, float x) {
      const uint32_t r = rank_of(e, x);
      if (r != HP_NONE && r >= rlo && r <= rhi) {
        const uint32_t k = tw_float_key(x);
        kmin = k < kmin ? k : kmin;
        if (small) {
          const uint32_t at = atomicAdd(&sh_n, 1u);
          if (at < HP_CAP) { cand_key[at] = k; cand_mass[at] = hp_fix(numer_of(e, x)); }
        }
      }
    });
    if (!small) {                                   // > HP_CAP scores within one rank: keep them all
      kmin = ~tw_wave_max_u32(~kmin);
      if (lane == 0) redf[wave] = __uint_as_float(kmin);
    }
    __syncthreads();
    TW_STAMP(8);
    if (wave == 0) {                                // one wave resolves; the others wait at the barrier
      if (small) {
        // lane x takes candidate x: mass of all candidates at least as large as it
        const uint32_t cn = sh_n < HP_CAP ? sh_n : HP_CAP;
        const uint32_t kx = lane < (int)cn ? cand_key[lane] : 0u;
        unsigned long long S = 0;
#pragma unroll 4
        for (uint32_t j = 0; j < cn; ++j) {
          const uint32_t kj = cand_key[j];
          const unsigned long long wj = cand_mass[j];
          S += kj >= kx ? wj : 0ull;
        }
        const uint32_t best = (lane < (int)cn && A + S >= target) ? kx : 0u;
        T = tw_wave_max_u32(best);
      } else {
        uint32_t r = __float_as_uint(redf[0]);
#pragma unroll
        for (int w = 1; w < NW; ++w) { const uint32_t y = __float_as_uint(redf[w]); r = y < r ? y : r; }
        T = r;
      }
      if (lane == 0) sh_T = T;
    }
    __syncthreads();
    T = sh_T;
    TW_STAMP(9);
  }

  // ---- LATE: the kernel's arguments, to be read again
  const auto late = [&] {
    if constexpr (LATE) {
      auto args = (const __attribute__((address_space(4))) HeadArgs*)__builtin_amdgcn_kernarg_segment_ptr();
      asm volatile("" : "+s"(args));
      return args;
    } else {
      return &a;
    }
  }();
  // ---- kept flags, count, optional ascending list; bitmap over token positions
  uint32_t cnt = 0, keep = 0;
  each([&](int e, float x) {
    const bool k = (INLDS ? (e >> 2) * 4 * NT + tid * 4 + (e & 3) : c0 + e) < N && tw_float_key(x) >= T;
    keep |= (k ? 1u : 0u) << e;
    cnt += k ? 1u : 0u;
  });
  uint32_t pos = 0;
  if (INLDS || !late->kept_idx) {
    const uint32_t wsumc = tw_wave_scan_u32(cnt);
    if (lane == 63 && wsumc) atomicAdd(&sh_kept, wsumc);
  } else {                                         // ordered positions need a scan over the block
    uint32_t total;
    const uint32_t incl = tw_block_scan_u32(cnt, ws32, &total);
    pos = incl - cnt;
    if (tid == 0) sh_kept = total;
  }
  if (TOK) {
    int32_t* out = late->kept_idx ? late->kept_idx + (long long)bh * late->kept_stride : nullptr;
#pragma unroll
    for (int e = 0; e < EPT; ++e) {
      if ((keep >> e) & 1u) {                       // kept => valid score => a token inside the sequence
        const int tok = pg[e % NPG];
        if ((uint32_t)tok < (uint32_t)(BWORDS * 32)) atomicOr(&bitmap[tok >> 5], 1u << (tok & 31));
        if (out) { if (pos < (uint32_t)late->kept_stride) out[pos] = tok; ++pos; }
      }
    }
  } else if (INLDS) {
    uint32_t run = 0;
#pragma unroll
    for (int v = 0; v < NPG; ++v) {
      const uint32_t mask = (keep >> (4 * v)) & 15u;
      const int tok0 = pg[v] * TW_PAGE + (tid * 4 & 15);
      if (mask && tok0 + 3 < BWORDS * 32) atomicOr(&bitmap[tok0 >> 5], mask << (tok0 & 31));
      if (late->kept_idx) {                             // ordered positions: the slots of v, of all threads, behind those of v - 1
        uint32_t total;
        const uint32_t c = __popc(mask), incl = tw_block_scan_u32(c, ws32, &total);
        pos = run + incl - c;
        int32_t* out = late->kept_idx + (long long)bh * late->kept_stride;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if ((mask >> e) & 1u) { if (pos < (uint32_t)late->kept_stride) out[pos] = tok0 + e; ++pos; }
        run += total;
      }
    }
  } else
#pragma unroll
  for (int v = 0; v < NPG; ++v) {
    constexpr int PB = EPT < 16 ? EPT : 16;        // slots of this thread inside page v
    const uint32_t mask = (keep >> (16 * v)) & ((1u << PB) - 1u);
    if (mask) {
      const int tok0 = pg[v] * TW_PAGE + (EPT < 16 ? (c0 & 15) : 0);
      if (tok0 + PB - 1 < BWORDS * 32) atomicOr(&bitmap[tok0 >> 5], mask << (tok0 & 31));
      if (late->kept_idx) {
        int32_t* out = late->kept_idx + (long long)bh * late->kept_stride;
#pragma unroll
        for (int e = 0; e < PB; ++e)
          if ((mask >> e) & 1u) { if (pos < (uint32_t)late->kept_stride) out[pos] = tok0 + e; ++pos; }
      }
    }
  }
  __syncthreads();
  uint32_t* bm = late->bitmaps + (long long)bh * late->words_stride;
#ifdef TW_FORMAL_ORDER
  // Measurement build: the hand-off written with the memory model's own pair - plain stores, a workgroup
  // barrier, one agent-scope acq_rel read-modify-write by thread 0 (release: everything the block wrote is
  // made visible to the agent first; acquire: nothing the reader loads afterwards may be stale).
  for (int i = tid; i < nwords; i += NT) bm[i] = bitmap[i];
  if (tid == 0) {
    uint32_t kc = sh_kept;
    if (late->kept_idx && kc > (uint32_t)late->kept_stride) { atomicOr(late->status, TW_STATUS_KEPT_TRUNCATED); kc = late->kept_stride; }
    late->kept_count[bh] = (int32_t)kc;
  }
  const int gi = b * a.Hkv + h / G;
  __syncthreads();
  if (tid == 0)
    sh_last = __hip_atomic_fetch_add(late->arrive + gi * TW_CTR, 1u, __ATOMIC_ACQ_REL, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(G - 1) ? 1u : 0u;
  __syncthreads();
#else
  // device-scope (write-through) stores: the group's last head reads these words from another CU
  for (int i = tid; i < nwords; i += NT) __hip_atomic_store(bm + i, bitmap[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  if (tid == 0) {
    uint32_t kc = sh_kept;
    if (late->kept_idx && kc > (uint32_t)late->kept_stride) { atomicOr(late->status, TW_STATUS_KEPT_TRUNCATED); kc = late->kept_stride; }
    late->kept_count[bh] = (int32_t)kc;
  }
  TW_STAMP(12);

  // ---- the last head of the KV head's group to get here turns the G bitmaps into the sorted union
  const int gi = b * a.Hkv + h / G;
  // Ordering without cache-wide fences: the bitmap words are stored and loaded with agent-scope atomics
  // (write-through stores, loads that bypass the caches that are not shared by all compute units), every
  // thread waits for the acknowledgement of its own stores (a workgroup barrier alone does not), the barrier
  // then collects the block, and only after it does thread 0 count the arrival.  The last head of the group
  // therefore finds every earlier head's words in place.  (The memory model's own form of this hand-off - plain
  // stores and an acq_rel counter, -DTW_FORMAL_ORDER - writes back and invalidates the whole L2 at every arrival.)
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
  if (tid == 0)
    sh_last = __hip_atomic_fetch_add(late->arrive + gi * TW_CTR, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) == (uint32_t)(G - 1) ? 1u : 0u;
  __syncthreads();
#endif
  if (!sh_last) return;
  TW_STAMP_IF(gi == 0, 14);
  if (tid == 0) __hip_atomic_store(late->arrive + gi * TW_CTR, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);   // ready for the next call
  // OR of the group's bitmaps into LDS (this block's own bitmap is no longer needed there): coalesced,
  // four words per thread and bitmap in flight
  const uint32_t* bmg = late->bitmaps + ((long long)(b * a.Hq + (h / G) * G)) * late->words_stride;
  for (int base = 0; base < nwords; base += 4 * NT) {
    uint32_t x[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      x[k] = 0;
      if (base + k * NT < nwords) {                  // block-uniform
        const int i = base + k * NT + tid;
        const int wi = i < nwords ? i : 0;
#pragma unroll
        for (int hh = 0; hh < G; ++hh)
#ifdef TW_FORMAL_ORDER
          x[k] |= bmg[(long long)hh * late->words_stride + wi];
#else
          x[k] |= __hip_atomic_load(bmg + (long long)hh * late->words_stride + wi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
#endif
      }
    }
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      const int i = base + k * NT + tid;
      if (i < nwords) bitmap[i] = x[k];
    }
  }
  __syncthreads();
  TW_STAMP_IF(gi == 0, 15);
  int32_t* uout = late->union_idx + (long long)gi * late->union_stride;
  uint32_t utotal;
  // (block-uniform choice: long sequences - more than two bitmap words per thread - take the wave-cooperative
  //  listing; with fewer words per thread the plain per-thread walk is as quick and needs fewer registers, which
  //  is what the 512-thread workgroups are short of)
  if (NT >= 1024 && nwords > 2 * NT) {
    // Wave w owns the contiguous words [w * wpw, (w + 1) * wpw) and takes them 64 at a time, one word per lane.  The
    // set bits of a round are listed either by every lane walking its own word (scattered kept tokens: few bits per
    // word) or, when fewer words are non-empty than the fullest word has bits (clustered heavy hitters: a few words
    // of 32), word by word with one lane per bit - two words at a time, one per half wave.
    const int wpw = (((nwords + NW - 1) / NW) + 63) & ~63;
    const int wbase = wave * wpw;
    uint32_t ucnt = 0;
    for (int r = 0; r < wpw; r += 64) {
      const int i = wbase + r + lane;
      ucnt += i < nwords ? __popc(bitmap[i]) : 0;
    }
    ucnt = tw_wave_scan_u32(ucnt);
    if (lane == 63) ws32[wave] = ucnt;
    __syncthreads();
    uint32_t run = 0;
    utotal = 0;
  #pragma unroll
    for (int w = 0; w < NW; ++w) { const uint32_t t = ws32[w]; run += w < wave ? t : 0u; utotal += t; }
    TW_STAMP_IF(gi == 0, 16);
    // positions staged in LDS and copied out coalesced when they fit (the usual case; block-uniform), else stored directly
    const bool staged = utotal <= (uint32_t)USTAGE;
    auto put = [&](uint32_t pos, int tok) {
      if (staged) ustage[pos] = tok;
      else if (pos < (uint32_t)late->union_stride) uout[pos] = tok;
    };
    for (int r = 0; r < wpw; r += 64) {               // wave-uniform trip count
      const int i = wbase + r + lane;
      uint32_t x = i < nwords ? bitmap[i] : 0u;
      const uint32_t c = __popc(x);
      const uint32_t incl = tw_wave_scan_u32(c);
      const uint32_t upos0 = run + incl - c;
      run += __shfl(incl, 63, 64);
      unsigned long long nz = __ballot(x != 0);
      if (nz == 0) continue;                           // wave-uniform
      const uint32_t maxc = tw_wave_max_u32(c);
      if ((uint32_t)__popcll(nz) * 2 >= maxc) {        // every lane its own word
        uint32_t upos = upos0;
        while (x) {
          const int bit = __ffs(x) - 1;
          x &= x - 1;
          put(upos++, i * 32 + bit);
        }
      } else {                                         // two non-empty words per step, one lane per bit
        const int half = lane >> 5, bit = lane & 31;
        while (nz) {                                   // wave-uniform
          const int s0 = __ffsll((long long)nz) - 1;
          nz &= nz - 1;
          int s1 = -1;
          if (nz) { s1 = __ffsll((long long)nz) - 1; nz &= nz - 1; }
          const int src = half ? s1 : s0;
          const uint32_t xw = (uint32_t)__shfl((int)x, src < 0 ? 0 : src, 64);
          const uint32_t ow = (uint32_t)__shfl((int)upos0, src < 0 ? 0 : src, 64);
          if (src >= 0 && ((xw >> bit) & 1u))
            put(ow + __popc(xw & ((1u << bit) - 1u)), (wbase + r + src) * 32 + bit);
        }
      }
    }
    if (staged) {
      __syncthreads();
      const uint32_t lim = utotal < (uint32_t)late->union_stride ? utotal : (uint32_t)late->union_stride;
      for (uint32_t i = tid; i < lim; i += NT) uout[i] = ustage[i];
    }
  } else {
    // thread t owns the contiguous words [t * wpt, (t + 1) * wpt): ascending output positions
    const int wpt = (nwords + NT - 1) / NT;
    const int w0 = tid * wpt, w1 = w0 + wpt < nwords ? w0 + wpt : nwords;
    uint32_t ucnt = 0;
    for (int i = w0; i < w1; ++i) ucnt += __popc(bitmap[i]);
    const uint32_t uincl = tw_block_scan_u32(ucnt, ws32, &utotal);
    TW_STAMP_IF(gi == 0, 16);
    uint32_t upos = uincl - ucnt;
    if (utotal <= (uint32_t)USTAGE) {               // block-uniform; the usual case
      // positions staged in LDS, then copied out coalesced: a dense word costs its thread 32 scattered
      // stores otherwise, one store instruction of the whole wave each (1.5 us of the kernel's tail)
      for (int i = w0; i < w1; ++i) {
        uint32_t x = bitmap[i];
        while (x) {
          const int bit = __ffs(x) - 1;
          x &= x - 1;
          ustage[upos++] = i * 32 + bit;
        }
      }
      __syncthreads();
      const uint32_t lim = utotal < (uint32_t)late->union_stride ? utotal : (uint32_t)late->union_stride;
      for (uint32_t i = tid; i < lim; i += NT) uout[i] = ustage[i];
    } else {
      for (int i = w0; i < w1; ++i) {
        uint32_t x = bitmap[i];
        while (x) {
          const int bit = __ffs(x) - 1;
          x &= x - 1;
          if (upos < (uint32_t)late->union_stride) uout[upos] = i * 32 + bit;
          ++upos;
        }
      }
    }
  }
  if (tid == 0) {
    if (utotal > (uint32_t)late->union_stride) { atomicOr(late->status, TW_STATUS_UNION_TRUNCATED); utotal = late->union_stride; }
    late->union_count[gi] = (int32_t)utotal;
  }
  TW_STAMP_IF(gi == 0, 13);
}

// ------------------------------------------------------------------ launches
int pages_per_wave(long long total_pages_all_rows, int count_bound) {
  // 4..64 pages per wave, at least ~8192 waves chip-wide (one per wave slot: measured at
  // 65536 candidate pages, 8 pages per wave beat 16 by 15 %; ragged batches whose bound is far
  // above the mean list length do best with long waves, fewer of which are empty)
  int pw = 64;
  while (pw > 4 && total_pages_all_rows / pw < 8192) pw >>= 1;
  while (pw > 4 && pw / 2 >= count_bound) pw >>= 1;
  return pw;
}

template <int NH, bool FULL>
void launch_score(const ScoreArgs& a, dim3 grid, bool dots, int bits, hipStream_t s) {
  // pages in flight per wave: 4, fewer when 8 heads share a page (register budget)
  if (bits == 2) {
    if (dots) TW_LAUNCH((int4_score_kernel<NH, FULL, true, 2, 2>), grid, dim3(256), 0, s, a);
    else      TW_LAUNCH((int4_score_kernel<NH, FULL, false, 2, 2>), grid, dim3(256), 0, s, a);
  } else if (bits == 8) {
    if (dots) TW_LAUNCH((int4_score_kernel<NH, FULL, true, 2, 8>), grid, dim3(256), 0, s, a);
    else      TW_LAUNCH((int4_score_kernel<NH, FULL, false, 2, 8>), grid, dim3(256), 0, s, a);
  }
  else if (dots) TW_LAUNCH((int4_score_kernel<NH, FULL, true, 2>), grid, dim3(256), 0, s, a);
  else if (NH < 8) TW_LAUNCH((int4_score_kernel<NH, FULL, false, 4>), grid, dim3(256), 0, s, a);
  else TW_LAUNCH((int4_score_kernel<NH, FULL, false, 2>), grid, dim3(256), 0, s, a);
}

bool score_uses_mfma(const TwDims& d, bool full) { return full && d.G >= 4 && d.bits == 4; }

int run_score(const twilight_kv_t* kv, const TwDims& d, const void* q, const int32_t* sel_pages,
              const int32_t* sel_count, int32_t max_sel, float* scores, int32_t* dots, uint32_t* arrive,
              uint32_t* headmax, hipStream_t s, const uint32_t* chmask = nullptr, unsigned long long* ghist = nullptr,
              const WhGrid* hgrid = nullptr) {
  ScoreArgs a;
  a.arrive = arrive; a.headmax = headmax; a.chmask = chmask; a.ghist = ghist; a.hgrid = hgrid;
  a.q = (const uint16_t*)q; a.sel_pages = sel_pages; a.sel_count = sel_count;
  a.page_table = kv->page_table; a.seq_lens = kv->seq_lens;
  a.kq_pool = (const uint4*)kv->kq_pool; a.kq_meta = (const uint32_t*)kv->kq_meta;
  a.scores = scores; a.dots = dots;
  a.Hq = d.Hq; a.Hkv = d.Hkv; a.max_pages = d.max_pages; a.max_sel = max_sel;
  a.pool_pages = d.pool_pages;
  const bool full = sel_pages == nullptr;
  const int bound = full ? d.max_pages : max_sel;
  a.cand_stride = bound * TW_PAGE;
  a.pw = pages_per_wave((long long)bound * d.batch * (full ? d.Hkv : d.Hq), bound);
#ifdef TW_TUNING                                 // tuning builds only: the shipped library reads no environment
  static const int pw_env = getenv("TW_INT4_PW") ? atoi(getenv("TW_INT4_PW")) : 0;
  static const int x_env = getenv("TW_INT4_X") ? atoi(getenv("TW_INT4_X")) : 0;
  static const bool valu_only = getenv("TW_INT4_VALU") && !ghist;   // vector-ALU kernel for every G
#else
  constexpr int pw_env = 0, x_env = 0;
  constexpr bool valu_only = false;
#endif
  // With the histogram every workgroup ends by adding its non-empty buckets to the heads' words, on which the row's other
  // workgroups queue: at most 96 to a row (1 x 32 heads x 100034 tokens: 391 to a row 54 us, 98 26, 49 23; 1 x 64 heads x
  // 26293: 103 to a row 30 us, 51 18; fewer than that leaves the chip idle: 2 x 32 x 85246 with 83 to a row 31 us, 42 37).
  if (ghist) while (a.pw < 64 && bound > 96 * 4 * a.pw) a.pw *= 2;
  if (pw_env >= 4 && pw_env <= 64) a.pw = pw_env;
  dim3 grid((bound + 4 * a.pw - 1) / (4 * a.pw), d.batch * (full ? d.Hkv : d.Hq));
  a.rotate = 0;
  if (!full) {
    // Per-head page lists: at most 8 pages per wave; rows of more than 8 chunks get a grid a multiple of 8 wide
    // (one column per XCD, see the kernel) and at most about 16384 workgroups - batches of many heads have
    // lists far shorter than the row bound, and their workgroups loop over the chunks beyond the grid
    if (!(pw_env >= 4 && pw_env <= 64) && a.pw > 8) a.pw = 8;
    int x = (bound + 4 * a.pw - 1) / (4 * a.pw);
    if (x > 8) {
      long long cap = 16384 / ((long long)d.batch * d.Hq);
      if (cap > x) cap = x;
      x = cap < 8 ? 8 : (int)(cap & ~7ll);
    }
    if (x_env > 0) x = x_env;
    grid.x = x;
    a.rotate = (x & 7) == 0 ? 1 : 0;
  }
  tw_prof_before(TW_K_INT4_SCORE, s);
  if (!full) launch_score<1, false>(a, grid, dots != nullptr, d.bits, s);
  else if (score_uses_mfma(d, full) && !valu_only) {              // matrix-core kernel: 4 or 8 heads share every page
    // 8 pages in flight per wave (the kernel needs few registers, so 4 to 7 waves per SIMD stay resident)
    if (d.G == 4) {
      if (dots) TW_LAUNCH((int4_score_mfma_kernel<1, true, 4>), grid, dim3(256), 0, s, a);
      else if (ghist) TW_LAUNCH((int4_score_mfma_kernel<1, false, 8, true>), grid, dim3(256), 0, s, a);
      else      TW_LAUNCH((int4_score_mfma_kernel<1, false, 8>), grid, dim3(256), 0, s, a);
    } else {
      if (dots) TW_LAUNCH((int4_score_mfma_kernel<2, true, 4>), grid, dim3(256), 0, s, a);
      else if (ghist) TW_LAUNCH((int4_score_mfma_kernel<2, false, 8, true>), grid, dim3(256), 0, s, a);
      else      TW_LAUNCH((int4_score_mfma_kernel<2, false, 8>), grid, dim3(256), 0, s, a);
    }
  } else switch (d.G) {
    case 1: launch_score<1, true>(a, grid, dots != nullptr, d.bits, s); break;
    case 2: launch_score<2, true>(a, grid, dots != nullptr, d.bits, s); break;
    case 4: launch_score<4, true>(a, grid, dots != nullptr, d.bits, s); break;
    default: launch_score<8, true>(a, grid, dots != nullptr, d.bits, s); break;
  }
  return tw_prof_after(s);
}


int run_row_sample(const twilight_kv_t* kv, const TwDims& d, const void* q, float p, WhGrid* hgrid, uint4* zero, long long zero16,
                   hipStream_t s) {
  SampleArgs a = {};
  a.s.q = (const uint16_t*)q; a.s.page_table = kv->page_table; a.s.seq_lens = kv->seq_lens;
  a.s.kq_pool = (const uint4*)kv->kq_pool; a.s.kq_meta = (const uint32_t*)kv->kq_meta;
  a.s.Hq = d.Hq; a.s.Hkv = d.Hkv; a.s.max_pages = d.max_pages; a.s.pool_pages = d.pool_pages;
  a.hgrid = hgrid; a.zero = zero; a.zero16 = zero16; a.heads = d.batch * d.Hq; a.p = p;
  tw_prof_before(TW_K_TOPP, s);
  TW_LAUNCH(row_sample_kernel, dim3(a.heads + SMP_ZERO_WGS), dim3(SMP_NT), 0, s, a);
  return tw_prof_after(s);
}

template <int NT, int EPT, bool TOK, int FUSE, int BITS>
void launch_topp_one(const HeadArgs& f, int G, dim3 grid, hipStream_t s) {
  switch (G) {
    case 1: TW_LAUNCH((topp_head_kernel<NT, EPT, 1, TOK, FUSE, BITS>), grid, dim3(NT), 0, s, f); break;
    case 2: TW_LAUNCH((topp_head_kernel<NT, EPT, 2, TOK, FUSE, BITS>), grid, dim3(NT), 0, s, f); break;
    case 4: TW_LAUNCH((topp_head_kernel<NT, EPT, 4, TOK, FUSE, BITS>), grid, dim3(NT), 0, s, f); break;
    default: TW_LAUNCH((topp_head_kernel<NT, EPT, 8, TOK, FUSE, BITS>), grid, dim3(NT), 0, s, f); break;
  }
}

// Register-resident top-p over rows of at most 8192 candidates (cand_stride = row bound).  Times in us, of the kernel alone.
//  - few heads: one 1024-thread workgroup per head (4 or 8 candidates per thread), or several (tw_prune_parts);
//  - more heads than CUs and rows of at most 4096 candidates: 512-thread workgroups, three to a CU, though two 1024-thread ones would
//    share a CU as well (64 registers with 4-bit codes, 52 on stored scores): three are at different phases, and each phase's barrier is
//    for half the waves.  With selection and scores inside, 1024 / 512 threads, by events: 4096 candidates of 1024 pages 288 heads 31.3 /
//    24.5, 512 35.5 / 25.6, 768 51.4 / 32.4, 1024 66.8 / 39.4, of 2048 pages 32.3 / 25.1, 35.8 / 27.0, 52.8 / 35.1, 68.1 / 45.5, of 8-bit
//    codes 512 heads 40.8 / 32.4; on stored scores 512 heads take 22.5 / 20.7, 1024 37.1 / 35.2, of token lists 19.4 / 18.6 and 35.0 / 32.0.  Selection and
//    scores inside: four to a CU, whose phases are longer, where that takes a round less and either the only one or the tables are short
//    (a thread of 512 has 8 of 4096 bounds, which the 64 registers hold worst).  Three and four to a CU, 4096 candidates of 1024 pages: 512
//    heads 31.2 / 33.5, 768 41.2 / 44.2, 1024 53.6 / 52.4, 1536 70.2 / 71.4, 2048 88.0 / 90.4, 4096 167.1 / 163.7; 2224 of 3750: 288 heads
//    25.6 / 29.6, 768 32.8 / 37.9, 1024 45.0 / 44.5, 2048 75.8 / 79.1; 4096 of 4096, 1024 heads: 58.0 / 59.7 (with 8-bit codes 76.2 / 82.0,
//    the one place where the line costs more than 3 %);
//  - rows of at most 2048 candidates (and, with the selection inside, at most 2048 pages): 512-thread workgroups with 4
//    candidates per thread, whatever the number of heads.  The kernel is a chain of block barriers; half the waves make
//    each shorter (32 heads x 1024 candidates 13.8 -> 11.7, 288 x 1024 23.2 -> 14.5), and with the LDS arrays sized
//    for the short rows four workgroups share a CU (64 registers; 2048 heads x 2048 candidates of 1024 pages 57.9 with 8 candidates per
//    thread, 53.0 with 4);
//  - rows of at most 1024 candidates and 1024 pages with more heads than CUs: 256-thread workgroups, eight to a CU (2048 heads x 256
//    candidates 34.2 -> 22.1, x 1024 40.2 -> 30.6, 288 x 256 12.8 -> 11.6; few heads, where it is no quicker, keep the 512 threads);
//  - more heads than CUs (behind a selection launch: than twice the CUs) with a bound above 4096 candidates, scoring inside:
//    512-thread workgroups with 16 candidates per thread, three (two) to a CU, for all heads - one's scoring streams while the others
//    are in their barriers (64 ragged sequences x 32 heads of up to 4096 pages: 180 with 1024 threads x 8, a workgroup per CU, 128 so;
//    8192 candidates: 10 x 32 heads 53.0 and 50.0, 16 x 32 62.6 and 52.3; 8 x 32, a workgroup per CU either way, 34.0 and 37.8.
//    the sequences with the most work first: twilight_select_prune);
//  - the same on stored scores (FUSE == 0): heads of at most 4096 candidates in a 512-thread launch of their own, the
//    longer ones in the 1024-thread launch.
// FUSE: the kernels score the candidates themselves (page lists).
template <bool TOK, int FUSE = 0, int BITS = 4>
int launch_topp(HeadArgs f, const TwDims& d, int cand_stride, hipStream_t s) {
  const dim3 grid(d.Hq * (FUSE == 3 ? f.parts : 1), d.batch);
  const long long heads = (long long)d.batch * d.Hq, cus = tw_num_cus();
  f.remap = (FUSE != 0 && ((long long)d.batch * d.Hkv) % 8 == 0) ? 1 : 0;
  f.n_above = -1; f.n_upto = cand_stride;
  // four workgroups of 8 candidates per thread to a CU instead of three
  const bool four = (heads + 4 * cus - 1) / (4 * cus) < (heads + 3 * cus - 1) / (3 * cus) && (heads <= 4 * cus || d.max_pages <= 1024);
  if constexpr (FUSE == 0) {
    if (cand_stride > 4096 && heads > 2 * cus) {
      f.n_upto = 4096;
      tw_prof_before(TW_K_TOPP, s);
      launch_topp_one<512, 8, TOK, FUSE, BITS>(f, d.G, grid, s);
      if (int e = tw_prof_after(s)) return e;
      f.n_above = 4096; f.n_upto = cand_stride;
    }
  }
  if constexpr (FUSE == 3) {
    tw_prof_before(TW_K_SELECT_SCORE_TOPP, s);
    launch_topp_one<1024, 8, TOK, FUSE, BITS>(f, d.G, grid, s);
    return tw_prof_after(s);
  } else {
  tw_prof_before(FUSE == 2 ? TW_K_SELECT_SCORE_TOPP : (FUSE == 1 ? TW_K_SCORE_TOPP : TW_K_TOPP), s);
  if (FUSE == 2 && heads > cus && cand_stride <= 1024 && d.max_pages <= 1024) launch_topp_one<FUSE == 2 ? 256 : 512, 4, TOK, FUSE, BITS>(f, d.G, grid, s);
  else if (cand_stride <= 2048 && (FUSE != 2 || d.max_pages <= 2048)) launch_topp_one<512, 4, TOK, FUSE, BITS>(f, d.G, grid, s);
  else if (FUSE == 2 && cand_stride <= 4096 && heads > cus && !four)
    launch_topp_one<512, 8, TOK, FUSE == 2 ? 4 : FUSE, BITS>(f, d.G, grid, s);
  else if (cand_stride <= 4096 && heads > cus) launch_topp_one<512, 8, TOK, FUSE, BITS>(f, d.G, grid, s);
  else if (cand_stride <= 4096) launch_topp_one<1024, 4, TOK, FUSE, BITS>(f, d.G, grid, s);
  else if (FUSE == 2 ? heads > cus : FUSE != 0 && heads > 2 * cus) launch_topp_one<512, FUSE != 0 ? 16 : 8, TOK, FUSE, BITS>(f, d.G, grid, s);
  else launch_topp_one<1024, 8, TOK, FUSE, BITS>(f, d.G, grid, s);
  return tw_prof_after(s);
  }
}

}  // namespace


// Channel-sparse estimate of every token of every sequence (the scoring half of the channel-sparse token selector):
// scores [b][Hq][max_pages * 16], tokens at or beyond the sequence's end -inf.
int tw_score_all_tokens_masked(const twilight_kv_t* kv, const TwDims& d, const void* q, const uint32_t* chmask, float* scores,
                               hipStream_t s) {
  return run_score(kv, d, q, nullptr, nullptr, 0, scores, nullptr, nullptr, nullptr, s, chmask);
}

int tw_prune_wide_init(const PruneWs& L, void* ws, bool full, hipStream_t s);
int tw_prune_wide(const TwDims& d, const PruneWs& L, void* ws, const twilight_kv_t* kv, const int32_t* sel_pages,
                  const int32_t* sel_count, int max_sel, int cand_stride, float p, int32_t* kept_count,
                  int32_t* kept_idx, int kept_stride, int32_t* union_count, int32_t* union_idx, int union_stride,
                  uint32_t* status, bool hist_done, hipStream_t s);

// Register-resident per-head kernel: per-head lists of at most 8192 candidates on sequences whose
// position bitmap fits in LDS; everything else takes the multi-workgroup path.
bool tw_prune_uses_head_kernel(const TwDims& d, bool full, int bound_pages) {
  return !full && bound_pages * TW_PAGE <= 1024 * 8 && (long long)d.max_pages * TW_PAGE <= HP_BITMAP_WORDS * 32ll;
}

PruneWs tw_prune_layout(const TwDims& d, int bound_pages, bool full) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t bh = (size_t)d.batch * d.Hq;
  PruneWs L;
  L.words_stride = (d.max_pages + 1) / 2;
  size_t o = 0;
  L.scores = o;  o += al(bh * (size_t)bound_pages * TW_PAGE * 4);
  const bool head = tw_prune_uses_head_kernel(d, full, bound_pages);
  L.headmax = o; o += head ? 256 : al(bh * HM_SLOTS * TW_CTR * 4);   // (the long-row path clears from here ...)
  L.arrive = o;  o += al((size_t)d.batch * d.Hkv * TW_CTR * 4);
  if (head) {                                                // the long-row buffers are not needed
    L.bitmaps = o; o += al(bh * (size_t)L.words_stride * 4);
    L.ghist = L.grid = L.range = L.sums = L.ucount = L.kdef = L.ulist = L.segcnt = o;
    L.total = o;
    return L;
  }
  L.ghist = o;   o += al(bh * WH_NB * 8);
  L.sums = o;    o += al(bh * WS_SUMS * 8);
  L.ucount = o;  o += al(bh * TW_CTR * 4);
  L.kdef = o;    o += al(bh * TW_CTR * 4);               // (... to here, with page lists to the bitmaps' end)
  L.bitmaps = o; o += al(bh * (size_t)L.words_stride * 4);
  L.grid = o;    o += al(bh * sizeof(WhGrid));
  L.range = o;   o += al(bh * 16);
  L.ulist = o;   o += al(bh * (size_t)WIDE_LIST_CAP * 8);
  L.segcnt = o;  o += al(bh * (size_t)((L.words_stride + 255) / 256) * 4);   // set bits per 256-word segment of a row's bitmap(s)
  L.total = o;
  return L;
}

#ifdef TW_PHASE_TIMING
extern "C" int twilight_debug_stamps_prune(unsigned long long* host_out) {
  return hipMemcpyFromSymbol(host_out, HIP_SYMBOL(tw_dbg_stamps), sizeof(unsigned long long) * 64) == hipSuccess ? 0 : -1;
}
#endif

extern "C" int twilight_int4_score(const twilight_kv_t* kv, const void* q, const int32_t* sel_pages,
                                   const int32_t* sel_count, int32_t max_sel, float* scores, int32_t* dots,
                                   void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !scores || !kv->kq_pool || !kv->kq_meta) return TW_EINVAL;
  if (sel_pages && (!sel_count || max_sel <= 0)) return TW_EINVAL;
  return run_score(kv, d, q, sel_pages, sel_count, max_sel, scores, dots, nullptr, nullptr, (hipStream_t)stream);
}

extern "C" int twilight_topp_prune(const twilight_kv_t* kv, const void* q, const int32_t* sel_pages,
                                   const int32_t* sel_count, int32_t max_sel, float p,
                                   int32_t* kept_count, int32_t* kept_idx, int32_t kept_stride,
                                   int32_t* union_count, int32_t* union_idx, int32_t union_stride,
                                   uint32_t* status, void* ws, size_t ws_bytes, void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !kept_count || !union_count || !union_idx || !status || !kv->kq_pool || !kv->kq_meta) return TW_EINVAL;
  if (sel_pages && (!sel_count || max_sel <= 0)) return TW_EINVAL;
  if (!(p > 0.f) || p > 1.f || union_stride <= 0 || (kept_idx && kept_stride <= 0)) return TW_EINVAL;
  const bool full = sel_pages == nullptr;
  const int bound = full ? d.max_pages : max_sel;
  if ((long long)bound * TW_PAGE > (1ll << 22)) return TW_EINVAL;   // fixed-point mass headroom
  if (!ws || ws_bytes < tw_prune_layout(d, bound, full).total) return TW_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  const int cand_stride = bound * TW_PAGE;
  const PruneWs L = tw_prune_layout(d, bound, full);
  float* scores = (float*)((char*)ws + L.scores);
  uint32_t* headmax = (uint32_t*)((char*)ws + L.headmax);
  uint32_t* arrive = (uint32_t*)((char*)ws + L.arrive);
  const bool use_head = tw_prune_uses_head_kernel(d, full, bound);

  const bool hist = !use_head && p < 1.0f && score_uses_mfma(d, full);
  if (hist) {                                    // the sample's launch clears what the next ones add to
    if (int e = run_row_sample(kv, d, q, p, (WhGrid*)((char*)ws + L.grid), (uint4*)headmax, (long long)((L.bitmaps - L.headmax) / 16), s))
      return e;
  } else if (!use_head) {
    if (int e = tw_prune_wide_init(L, ws, full, s)) return e;  // clears headmax before the scoring kernel folds into it
  }
  unsigned long long* const ghist = hist ? (unsigned long long*)((char*)ws + L.ghist) : nullptr;
  WhGrid* const hgrid = hist ? (WhGrid*)((char*)ws + L.grid) : nullptr;
  if (int e = run_score(kv, d, q, sel_pages, sel_count, max_sel, scores, nullptr, use_head ? arrive : nullptr,
                        use_head ? nullptr : headmax, s, nullptr, ghist, hgrid)) return e;
  if (!use_head)
    return tw_prune_wide(d, L, ws, kv, sel_pages, sel_count, max_sel, cand_stride, p, kept_count, kept_idx, kept_stride,
                         union_count, union_idx, union_stride, status, hist, s);

  // per-head page lists short enough for registers and sequences that fit the LDS bitmap: one
  // launch does top-p per head and, in the last head of each group to finish, the group's union
  {
    const int words_stride = L.words_stride;
    uint32_t* bitmaps = (uint32_t*)((char*)ws + L.bitmaps);
    HeadArgs f;
    f.scores = scores; f.sel_pages = sel_pages; f.sel_count = sel_count; f.seq_lens = kv->seq_lens;
    f.kept_count = kept_count; f.kept_idx = kept_idx; f.bitmaps = bitmaps; f.arrive = arrive;
    f.union_count = union_count; f.union_idx = union_idx; f.status = status;
    f.Hq = d.Hq; f.Hkv = d.Hkv; f.max_pages = d.max_pages; f.max_sel = max_sel; f.cand_stride = cand_stride;
    f.kept_stride = kept_stride; f.words_stride = words_stride; f.union_stride = union_stride; f.p = p;
    f.q = nullptr; f.page_table = nullptr; f.kq_pool = nullptr; f.kq_meta = nullptr; f.pool_pages = 0;
    f.bounds = nullptr; f.budget = nullptr; f.sel_pages_w = nullptr; f.sel_count_w = nullptr; f.scores_w = nullptr; f.parts = 1; f.ordered = 0;
    return launch_topp<false>(f, d, cand_stride, s);
  }
}

// Pruner over per-head page lists with the scoring done inside the top-p kernel (one launch).  The arrival
// counters at `ws` + layout.arrive must be zero: a kernel earlier on the stream clears them.
// bounds != nullptr: the kernel also selects the head's pages from the bounds of all pages ([b][Hq][max_pages],
// with the budgets) and writes the lists to sel_pages / sel_count; else it reads the lists from there.
bool tw_prune_fused_ok(const TwDims& d, int max_sel, bool with_select) {
  if (max_sel <= 0 || !tw_prune_uses_head_kernel(d, false, max_sel) || (d.bits != 4 && !with_select)) return false;
  return !with_select || d.max_pages <= 4096;      // the selection's keys share the kernel's LDS staging array
}
// Workgroups per head when it is to be split (see topp_head_kernel, FUSE == 3), 1: not.  As many as give every CU one, for
// lists above 4096 candidates on at most half as many heads as CUs (selector and pruner, us, against launches of their own: 1 x 32 heads
// x 4096 pages x 8192 candidates 33.6 -> 31.5, 2 x 32 41.1 -> 37.1, 4 x 32 49.7 -> 45.8).  Shorter lists lose: the hand-off costs 1.4 us and reading the
// scores back 2 (32 heads x 4096 candidates 19.9 us in one workgroup each, 21.4 split; 64 x 2000 14.4 and 20.1).
int tw_prune_parts(const TwDims& d, int max_sel) {
  const long long heads = (long long)d.batch * d.Hq;
  if (max_sel <= 0 || !tw_prune_uses_head_kernel(d, false, max_sel) || d.max_pages > 8192) return 1;
  if (max_sel * TW_PAGE <= 4096 || 2 * heads > tw_num_cus()) return 1;
  const long long fit = tw_num_cus() / heads;
  return (int)(fit > 8 ? 8 : fit);
}
int tw_prune_fused(const twilight_kv_t* kv, const TwDims& d, const void* q, const float* bounds, const int32_t* budget,
                   int32_t* sel_pages, int32_t* sel_count, int32_t max_sel, float p, int32_t* kept_count, int32_t* kept_idx,
                   int32_t kept_stride, int32_t* union_count, int32_t* union_idx, int32_t union_stride,
                   uint32_t* status, void* ws, int parts, bool ordered, hipStream_t s) {
  const PruneWs L = tw_prune_layout(d, max_sel, false);
  HeadArgs f;
  f.parts = parts;
  f.scores = f.scores_w = parts > 1 ? (float*)((char*)ws + L.scores) : nullptr; f.sel_pages = sel_pages; f.sel_count = sel_count; f.seq_lens = kv->seq_lens;
  f.kept_count = kept_count; f.kept_idx = kept_idx; f.bitmaps = (uint32_t*)((char*)ws + L.bitmaps);
  f.arrive = (uint32_t*)((char*)ws + L.arrive);
  f.union_count = union_count; f.union_idx = union_idx; f.status = status;
  f.Hq = d.Hq; f.Hkv = d.Hkv; f.max_pages = d.max_pages; f.max_sel = max_sel; f.cand_stride = max_sel * TW_PAGE;
  f.kept_stride = kept_stride; f.words_stride = L.words_stride; f.union_stride = union_stride; f.p = p;
  f.q = (const uint16_t*)q; f.page_table = kv->page_table; f.kq_pool = (const uint4*)kv->kq_pool;
  f.kq_meta = (const uint32_t*)kv->kq_meta; f.pool_pages = d.pool_pages;
  f.bounds = bounds; f.budget = budget; f.sel_pages_w = sel_pages; f.sel_count_w = sel_count;
  f.ordered = ordered ? 1 : 0;
  if (parts > 1 && d.bits == 8) return launch_topp<false, 3, 8>(f, d, max_sel * TW_PAGE, s);
  if (parts > 1 && d.bits == 2) return launch_topp<false, 3, 2>(f, d, max_sel * TW_PAGE, s);
  if (parts > 1) return launch_topp<false, 3>(f, d, max_sel * TW_PAGE, s);
  if (bounds && d.bits == 8) return launch_topp<false, 2, 8>(f, d, max_sel * TW_PAGE, s);
  if (bounds && d.bits == 2) return launch_topp<false, 2, 2>(f, d, max_sel * TW_PAGE, s);
  if (bounds) return launch_topp<false, 2>(f, d, max_sel * TW_PAGE, s);
  return launch_topp<false, 1>(f, d, max_sel * TW_PAGE, s);
}

// ------------------------------------------------------------------ token-list candidates
static int tw_check_tokens(const TwDims& d, int32_t max_cand) {
  if (max_cand <= 0 || (max_cand & 15) || max_cand > 1024 * 8) return TW_EINVAL;
  if ((long long)d.max_pages * TW_PAGE > HP_BITMAP_WORDS * 32ll) return TW_EINVAL;
  return TW_OK;
}

PruneWs tw_prune_layout_tokens(const TwDims& d, int max_cand) {
  auto al = [](size_t x) { return (x + 255) & ~(size_t)255; };
  const size_t bh = (size_t)d.batch * d.Hq;
  PruneWs L;
  L.words_stride = (d.max_pages + 1) / 2;
  size_t o = 0;
  L.scores = o;  o += al(bh * (size_t)max_cand * 4);
  L.headmax = o;
  L.arrive = o;  o += al((size_t)d.batch * d.Hkv * TW_CTR * 4);
  L.bitmaps = o; o += al(bh * (size_t)L.words_stride * 4);
  L.ghist = L.grid = L.range = L.sums = L.ucount = L.kdef = L.ulist = L.segcnt = o;
  L.total = o;
  return L;
}

static int run_score_tokens(const twilight_kv_t* kv, const TwDims& d, const void* q, const int32_t* cand_tokens,
                            const int32_t* cand_count, int32_t max_cand, float* scores, int32_t* dots,
                            uint32_t* arrive, hipStream_t s) {
  ScoreArgs a;
  a.arrive = arrive; a.headmax = nullptr; a.chmask = nullptr; a.ghist = nullptr; a.hgrid = nullptr;
  a.q = (const uint16_t*)q; a.sel_pages = cand_tokens; a.sel_count = cand_count;
  a.page_table = kv->page_table; a.seq_lens = kv->seq_lens;
  a.kq_pool = (const uint4*)kv->kq_pool; a.kq_meta = (const uint32_t*)kv->kq_meta;
  a.scores = scores; a.dots = dots;
  a.Hq = d.Hq; a.Hkv = d.Hkv; a.max_pages = d.max_pages; a.max_sel = max_cand; a.cand_stride = max_cand; a.pw = 0; a.rotate = 0;
  a.pool_pages = d.pool_pages;
  // grid as for page lists: rows of more than 8 chunks get a width that is a multiple of 8, cut so that the
  // launch stays near 16384 workgroups; the workgroups loop over the chunks beyond it
  int x = (max_cand + 255) / 256;
  if (x > 8) {
    long long cap = 16384 / ((long long)d.batch * d.Hq);
    if (cap > x) cap = x;
    x = cap < 8 ? 8 : (int)(cap & ~7ll);
  }
  a.rotate = (x & 7) == 0 ? 1 : 0;
  const dim3 grid(x, d.batch * d.Hq);
  tw_prof_before(TW_K_INT4_SCORE, s);
  if (d.bits == 2) {
    if (dots) TW_LAUNCH((int4_score_tokens_kernel<true, 2>), grid, dim3(256), 0, s, a);
    else      TW_LAUNCH((int4_score_tokens_kernel<false, 2>), grid, dim3(256), 0, s, a);
  } else if (d.bits == 8) {
    if (dots) TW_LAUNCH((int4_score_tokens_kernel<true, 8>), grid, dim3(256), 0, s, a);
    else      TW_LAUNCH((int4_score_tokens_kernel<false, 8>), grid, dim3(256), 0, s, a);
  } else {
    if (dots) TW_LAUNCH((int4_score_tokens_kernel<true, 4>), grid, dim3(256), 0, s, a);
    else      TW_LAUNCH((int4_score_tokens_kernel<false, 4>), grid, dim3(256), 0, s, a);
  }
  return tw_prof_after(s);
}

extern "C" int twilight_int4_score_tokens(const twilight_kv_t* kv, const void* q, const int32_t* cand_tokens,
                                          const int32_t* cand_count, int32_t max_cand, float* scores, int32_t* dots,
                                          void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !scores || !cand_tokens || !cand_count || !kv->kq_pool || !kv->kq_meta) return TW_EINVAL;
  if (int e = tw_check_tokens(d, max_cand)) return e;
  return run_score_tokens(kv, d, q, cand_tokens, cand_count, max_cand, scores, dots, nullptr, (hipStream_t)stream);
}

extern "C" int twilight_topp_prune_tokens(const twilight_kv_t* kv, const void* q, const int32_t* cand_tokens,
                                          const int32_t* cand_count, int32_t max_cand, float p,
                                          int32_t* kept_count, int32_t* kept_idx, int32_t kept_stride,
                                          int32_t* union_count, int32_t* union_idx, int32_t union_stride,
                                          uint32_t* status, void* ws, size_t ws_bytes, void* stream) {
  TwDims d;
  if (int e = tw_check_kv(kv, &d)) return e;
  if (!q || !cand_tokens || !cand_count || !kept_count || !union_count || !union_idx || !status || !kv->kq_pool || !kv->kq_meta)
    return TW_EINVAL;
  if (!(p > 0.f) || p > 1.f || union_stride <= 0 || (kept_idx && kept_stride <= 0)) return TW_EINVAL;
  if (int e = tw_check_tokens(d, max_cand)) return e;
  const PruneWs L = tw_prune_layout_tokens(d, max_cand);
  if (!ws || ws_bytes < L.total) return TW_EWORKSPACE;
  hipStream_t s = (hipStream_t)stream;
  float* scores = (float*)((char*)ws + L.scores);
  uint32_t* arrive = (uint32_t*)((char*)ws + L.arrive);
  if (int e = run_score_tokens(kv, d, q, cand_tokens, cand_count, max_cand, scores, nullptr, arrive, s)) return e;
  HeadArgs f;
  f.scores = scores; f.sel_pages = cand_tokens; f.sel_count = cand_count; f.seq_lens = kv->seq_lens;
  f.kept_count = kept_count; f.kept_idx = kept_idx; f.bitmaps = (uint32_t*)((char*)ws + L.bitmaps); f.arrive = arrive;
  f.union_count = union_count; f.union_idx = union_idx; f.status = status;
  f.Hq = d.Hq; f.Hkv = d.Hkv; f.max_pages = d.max_pages; f.max_sel = max_cand; f.cand_stride = max_cand;
  f.kept_stride = kept_stride; f.words_stride = L.words_stride; f.union_stride = union_stride; f.p = p;
  f.q = nullptr; f.page_table = nullptr; f.kq_pool = nullptr; f.kq_meta = nullptr; f.pool_pages = 0;
  f.bounds = nullptr; f.budget = nullptr; f.sel_pages_w = nullptr; f.sel_count_w = nullptr; f.scores_w = nullptr; f.parts = 1; f.ordered = 0;
  return launch_topp<true>(f, d, max_cand, s);
}
