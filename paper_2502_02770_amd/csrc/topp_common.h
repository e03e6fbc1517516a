// Pieces shared by the top-p kernels (register-resident per-head path and
// the multi-workgroup path for long candidate rows).
#pragma once
#include "tw_common.h"

constexpr uint32_t kKeyNegInf = 0x007FFFFFu;   // tw_float_key(-inf)

constexpr int HP_NB = 512;                     // histogram buckets per pass
constexpr uint32_t HP_FINE_END = 1u << 25;     // ranks below this (8 logits under the max) get the fine first pass
constexpr uint32_t HP_NONE = 0xFFFFFFFFu;      // rank of a score that takes no part (invalid slot or zero mass)
// Words that many workgroups update with atomics (head maxima, counters) sit 128 bytes apart:
// atomics to one cache line are served one after the other, whatever word they address.
constexpr int TW_CTR = 32;                     // stride in 32-bit words
// The long-row path's per-head maximum is folded by every scoring workgroup: spread over this
// many words per head (workgroup x folds into word x % HM_SLOTS); readers take the max of them.
constexpr int HM_SLOTS = 32;

// Long-row path: histogram over the scores of a row (wh_bucket below), sums per head, list capacity.
constexpr int WH_HALF = 640, WH_NB = 2 * WH_HALF;
constexpr int WH_LDS = WH_NB + 16;             // stride of one head's histogram in LDS: four heads' equal buckets on different banks
constexpr int WS_SUMS = 16;                    // 64-bit words per head (128 bytes)
constexpr int WIDE_LIST_CAP = 8192;

// Workspace of twilight_topp_prune (byte offsets).  Both paths use scores,
// headmax, bitmaps, arrive; the rest belongs to the long-row path.
struct PruneWs {
  size_t scores, headmax, bitmaps, arrive, ghist, grid, range, sums, ulist, ucount, kdef, segcnt, total;
  int words_stride;       // bitmap words per head
};
PruneWs tw_prune_layout(const TwDims& d, int bound_pages, bool full);
PruneWs tw_prune_layout_tokens(const TwDims& d, int max_cand);   // token-list candidates (register-resident path only)

int tw_score_all_tokens_masked(const twilight_kv_t* kv, const TwDims& d, const void* q, const uint32_t* chmask, float* scores,
                               hipStream_t s);

// The pruner with the scoring - and, with `bounds`, the page selection - inside the per-head top-p kernel (per-head
// page lists, 4-bit codes, rows short enough for registers: tw_prune_fused_ok).  ws = a TW_WS_PRUNE workspace for
// this max_sel whose arrival counters (tw_prune_layout(d, max_sel, false).arrive, batch * Hkv * TW_CTR words) a
// kernel earlier on the stream has cleared.
bool tw_prune_fused_ok(const TwDims& d, int max_sel, bool with_select);
int tw_prune_fused(const twilight_kv_t* kv, const TwDims& d, const void* q, const float* bounds, const int32_t* budget,
                   int32_t* sel_pages, int32_t* sel_count, int32_t max_sel, float p, int32_t* kept_count, int32_t* kept_idx,
                   int32_t kept_stride, int32_t* union_count, int32_t* union_idx, int32_t union_stride,
                   uint32_t* status, void* ws, int parts, bool ordered, hipStream_t s);
// Batches of more heads than run at once, of at most TW_ORDER_MAX sequences: the kernel that clears the counters leaves the order in
// which their heads are to be dispatched, place i's sequence in a spare word of the counters' lines.
constexpr int TW_ORDER_MAX = 256;
int tw_prune_parts(const TwDims& d, int max_sel);   // workgroups per head of the split form, which selects its pages itself; 1: not split

#ifdef __HIPCC__
__device__ __forceinline__ long long tw_order_word(int i, int Hkv) { return (long long)i * Hkv * TW_CTR + TW_CTR - 1; }

// softmax numerator e in [0, 1] -> floor(e * 2^40), exactly: the top 8 bits and the remaining 32
// bits are taken by two float -> integer truncations (every step below is exact in fp32: scaling by
// a power of two, the integer part of a value below 2^9, and the difference of the two)
__device__ __forceinline__ unsigned long long hp_fix(float e) {
  const float t = e * 256.0f;
  const uint32_t hi = (uint32_t)t;
  const float rem = t - (float)hi;
  const uint32_t lo = (uint32_t)(rem * 4294967296.0f);
  return ((unsigned long long)hi << 32) | lo;
}
constexpr float HP_REACH = 27.5f;              // logits below the max at which a score stops taking part
// rank of a score: distance to the max logit in 2^-22 units; HP_NONE when the score is
// invalid or more than 27.5 logits below the max (its 2^-40 fixed-point mass is at most one unit there)
__device__ __forceinline__ uint32_t hp_rank_only(float m, float s) {
  const float d = __fsub_rn(m, s);
  return d < HP_REACH ? (uint32_t)(d * 4194304.f) : HP_NONE;
}
__device__ __forceinline__ float hp_numer(float m, float s) { return __expf(-__fsub_rn(m, s)); }
// mass the kept scores have to reach: p of the total, at least one unit
__device__ __forceinline__ unsigned long long hp_target(float p, unsigned long long Z) {
  const double t = ceil((double)p * (double)Z);
  const unsigned long long target = t < 1.0 ? 1ull : (unsigned long long)t;
  return target > Z ? Z : target;
}
// Where a row's histogram is fine: buckets are laid out over t = (s - ref) / scale.
struct WhGrid { float ref, scale; };
// Bucket of t, larger scores first.  64 buckets per doubling of |t| + 1/2 - 1/128 wide at 0, 1/64 from 0.5, 1/32 from 1.5,
// and so on out to 511 - so a grid that was laid around the threshold by a sample leaves few scores in the bucket the
// threshold falls into, and one that was not still tells scores apart to 1/64 of their distance from it.
// A score's weight relative to the bucket's upper edge, exp(-(distance to it)), comes in units of 2^-19: a bucket's sum
// is its mass to within the rounding of these (the 4096 scores of a scoring workgroup fit 32 bits).  lscale =
// scale * log2(e).  In the outermost buckets the weight is relative to an edge further out.
__device__ __forceinline__ int wh_bucket(float t, float lscale, uint32_t* q) {
  const float a = fabsf(t) + 0.5f;
  const uint32_t ab = __float_as_uint(a), near = ab & 0xFFFE0000u;
  uint32_t u = (ab - 0x3F000000u) >> 17;
  u = u < WH_HALF - 1u ? u : WH_HALF - 1u;
  const bool neg = t < 0.f;
  const float edge = __uint_as_float(neg ? near : near + 0x20000u);
  *q = (uint32_t)__builtin_amdgcn_exp2f(__builtin_fmaf(-fabsf(a - edge), lscale, 19.0f));
  return neg ? WH_HALF + (int)u : WH_HALF - 1 - (int)u;
}
// |t| at which bucket u (from 0) of either half begins
__device__ __forceinline__ float wh_edge(int u) { return __uint_as_float(0x3F000000u + ((uint32_t)u << 17)) - 0.5f; }
// The grid for a row's top-p threshold, from sums over a sample of its scores, weighted by w = exp(s - max of the
// sample): the scores that carry the mass have mean sws / sw, and p = 0.8 .. 0.99 of it ends one or two deviations below.
// The scale is a quarter of the deviation, but at least 1/8 logit: the grid then reaches 64 logits to either side.
__device__ __forceinline__ WhGrid wh_grid(float sw, float sws, float swss) {
  WhGrid g;
  g.ref = 0.f; g.scale = 1.f;
  if (sw > 0.f) {
    const float mean = sws / sw, var = swss / sw - mean * mean;
    if (var >= 0.f && var < 1.0e6f && fabsf(mean) < 1.0e30f) {
      g.scale = fmaxf(0.25f * sqrtf(var), 0.125f);
      g.ref = mean - 1.3f * sqrtf(var);
    }
  }
  return g;
}
__device__ __forceinline__ uint32_t hp_rank(float m, float s, float* e_out) {
  *e_out = hp_numer(m, s);
  return hp_rank_only(m, s);
}
#endif
