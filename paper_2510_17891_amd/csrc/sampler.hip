// Stand-alone Gumbel-max sampling kernels (logits in memory) and the merge stage shared with the fused path.
// The arithmetic contract lives in sampler_device.h.  The log-probability log softmax(z/T)[token] is accumulated
// in fp32 (tolerance, not bit-exact).
#include <algorithm>
#include <mutex>
#include <type_traits>

#include "../../include/rl.h"
#include "cut_plan.h"
#include "kernels.h"
#include "sampler_device.h"

namespace rl {

namespace {

// Stage 1: grid (tiles, rows); each block scans kSampleTile vocabulary entries of one row of fp32 logits.
__global__ __launch_bounds__(256) void sample_stage1_kernel(const float* __restrict__ logits, int V,
                                                            const RowMeta* __restrict__ rows, int pos_offset, float inv_t,
                                                            int greedy, uint32_t seed_lo, uint32_t seed_hi,
                                                            const int32_t* __restrict__ forced, float* __restrict__ forced_z,
                                                            float* __restrict__ part, int n_tiles) {
  __shared__ float sh_y[4], sh_z[4], sh_m[4], sh_s[4];
  __shared__ int sh_i[4];
  const int tile = blockIdx.x, r = blockIdx.y;
  const RowMeta rm = rows[r];
  const uint32_t pos = (uint32_t)(rm.pos + pos_offset), seq = (uint32_t)rm.seq;
  const float* z = logits + (size_t)r * V;
  const int f = forced ? forced[r] : -1;
  Best best{-INFINITY, -1, 0.f};
  float m = -INFINITY, s = 0.f;
  const int i_end = min(V, (tile + 1) * kSampleTile);
  for (int i0 = tile * kSampleTile + threadIdx.x * 4; i0 < i_end; i0 += 256 * 4) {
    const float zs[4] = {z[i0], z[i0 + 1], z[i0 + 2], z[i0 + 3]};  // V and the tile are multiples of four
    uint32_t rnd[4] = {0, 0, 0, 0};
    if (!greedy) philox4x32_10((uint32_t)i0 >> 2, pos, seq, 0u, seed_lo, seed_hi, rnd);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int i = i0 + e;
      const float zi = zs[e];
      const float y = greedy ? zi : __fmaf_rn(zi, inv_t, gumbel(rnd[e]));
      best = better(best, Best{y, i, zi});
      lse_add(m, s, zi * inv_t);
      if (i == f) forced_z[r] = zi;
    }
  }
  each_mask([&](int o) __attribute__((always_inline)) {
    best = best_of_lanes(best, o);
    lse_merge_lanes(m, s, o);
  });
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) { sh_y[wave] = best.y; sh_i[wave] = best.idx; sh_z[wave] = best.z; sh_m[wave] = m; sh_s[wave] = s; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < 4; ++w) {
      best = better(best, Best{sh_y[w], sh_i[w], sh_z[w]});
      lse_merge(m, s, sh_m[w], sh_s[w]);
    }
    float* p = part + ((size_t)r * n_tiles + tile) * kSamplePartFloats;
    *(float4*)p = make_float4(best.y, __int_as_float(best.idx), best.z, 0.f);
    *(float4*)(p + 4) = make_float4(m, s, 0.f, 0.f);
  }
}

constexpr int kSampleRowMax = 8192;
// Both stages in one block per row, for vocabularies of a few thousand entries, where each launch lasts as long as its chain of
// round trips whatever it does.  Kernel times, two launches -> one: 4 rows of 4096 entries 9.5 -> 5.9 us, 1 row of 8192 8.4 ->
// 7.2, 1024 rows of 8192 27.5 -> 23.  At 12288 entries a row or two take as long either way, at 16384 8.4 in two launches and
// 11.0 in one.  Which kernel runs depends on the vocabulary alone, and so do a row's bits: the loads need no alignment
// beyond that of a float.
__global__ __launch_bounds__(1024) void sample_row_kernel(const float* __restrict__ logits, int V, const RowMeta* __restrict__ rows,
                                                          int pos_offset, float inv_t, int greedy, uint32_t seed_lo, uint32_t seed_hi,
                                                          const int32_t* __restrict__ forced, int32_t* __restrict__ out_tok,
                                                          float* __restrict__ out_lp, int32_t* __restrict__ last_tok) {
  __shared__ float sh_y[16], sh_z[16], sh_m[16], sh_s[16], sh_forced;
  __shared__ int sh_i[16];
  const int r = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const float* z = logits + (size_t)r * V;
  const int first = threadIdx.x * 4, step = blockDim.x * 4;
  const auto load = [&](int i) __attribute__((always_inline)) { return make_float4(z[i], z[i + 1], z[i + 2], z[i + 3]); };  // one load
  float4 v = load(first < V ? first : 0);  // V is a multiple of four
  const RowMeta rm = rows[r];
  const uint32_t pos = (uint32_t)(rm.pos + pos_offset), seq = (uint32_t)rm.seq;
  const int f = forced ? forced[r] : -1;
  Best best{-INFINITY, -1, 0.f};
  float m = -INFINITY, s = 0.f;
  for (int i0 = first; i0 < V; i0 += step) {
    const float zs[4] = {v.x, v.y, v.z, v.w};
    if (i0 + step < V) v = load(i0 + step);
    uint32_t rnd[4] = {0, 0, 0, 0};
    if (!greedy) philox4x32_10((uint32_t)i0 >> 2, pos, seq, 0u, seed_lo, seed_hi, rnd);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const float y = greedy ? zs[e] : __fmaf_rn(zs[e], inv_t, gumbel(rnd[e]));
      best = better(best, Best{y, i0 + e, zs[e]});
      lse_add(m, s, zs[e] * inv_t);
      if (i0 + e == f) sh_forced = zs[e];
    }
  }
  const auto merge = [&](int o) __attribute__((always_inline)) {
    best = best_of_lanes(best, o);
    lse_merge_lanes(m, s, o);
  };
  each_mask(merge);
  if (lane == 0) { sh_y[wave] = best.y; sh_i[wave] = best.idx; sh_z[wave] = best.z; sh_m[wave] = m; sh_s[wave] = s; }
  __syncthreads();
  if (wave != 0) return;
  const bool there = lane < (int)(blockDim.x >> 6);
  const int w = lane & 15;
  best = there ? Best{sh_y[w], sh_i[w], sh_z[w]} : Best{-INFINITY, -1, 0.f};
  m = there ? sh_m[w] : -INFINITY;
  s = there ? sh_s[w] : 0.f;
  each_mask<8>(merge);
  if (lane != 0) return;
  int tok = best.idx < 0 ? 0 : best.idx;  // idx < 0 only when every score was NaN
  float zt = best.z;
  if (f >= 0 && f < V) { tok = f; zt = sh_forced; }
  out_tok[r] = tok;
  if (last_tok != nullptr) last_tok[rm.seq] = tok;
  out_lp[r] = zt * inv_t - (m + logf(s));
}

// Stage 2: one block per row merges the tile partials and emits token and log-probability: 1024 threads, or one wave
// where there are at most 64 partials (the same merges: further waves would hold nothing).
__global__ __launch_bounds__(1024) void sample_stage2_kernel(const float* __restrict__ part, int n_tiles, int V,
                                                             const int32_t* __restrict__ forced,
                                                             const float* __restrict__ forced_z, float inv_t,
                                                             int32_t* __restrict__ out_tok, float* __restrict__ out_lp,
                                                             const RowMeta* __restrict__ rows, int32_t* __restrict__ last_tok) {
  __shared__ float sh_y[16], sh_z[16], sh_m[16], sh_s[16];
  __shared__ int sh_i[16];
  const int r = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  Best best{-INFINITY, -1, 0.f};
  float m = -INFINITY, s = 0.f;
  for (int t = threadIdx.x; t < n_tiles; t += blockDim.x) {
    const float* p = part + ((size_t)r * n_tiles + t) * kSamplePartFloats;
    const float4 a = *(const float4*)p;
    const float4 b = *(const float4*)(p + 4);
    best = better(best, Best{a.x, __float_as_int(a.y), a.z});
    lse_merge(m, s, b.x, b.y);
  }
  each_mask([&](int o) __attribute__((always_inline)) {
    best = best_of_lanes(best, o);
    lse_merge_lanes(m, s, o);
  });
  if (lane == 0) { sh_y[wave] = best.y; sh_i[wave] = best.idx; sh_z[wave] = best.z; sh_m[wave] = m; sh_s[wave] = s; }
  __syncthreads();
  if (threadIdx.x == 0) {
    for (int w = 1; w < (int)(blockDim.x >> 6); ++w) {
      best = better(best, Best{sh_y[w], sh_i[w], sh_z[w]});
      lse_merge(m, s, sh_m[w], sh_s[w]);
    }
    int tok = best.idx < 0 ? 0 : best.idx;  // idx < 0 only when every score was NaN
    float zt = best.z;
    if (forced != nullptr && forced[r] >= 0 && forced[r] < V) { tok = forced[r]; zt = forced_z[r]; }
    out_tok[r] = tok;
    if (last_tok != nullptr) last_tok[rows[r].seq] = tok;  // what the sequence is fed next when the caller passes no tokens
    out_lp[r] = zt * inv_t - (m + logf(s));
  }
}


// ------------------------------------------------------------------------------------------------
// Truncated sampling: the top-k / top-p cut of every row (the last kept token of the order) and the draw from what is
// left, in three passes over the logits.
//   1. cut_range: largest and smallest logit of the row, how far below the largest its bulk lies, and the largest logit of
//      every unit of 256, by which pass 3 leaves out what lies behind the cut.
//   2. cut_hist: count or integer mass per bin, the bins being steps of the logit below the largest one.  A mass has
//      kCutBins equal steps over the 22 / inv_t in which weights are not zero.  A count has the finest steps over four
//      times the distance to the largest minimum of four neighbouring logits (or 64 times that of two, where that is less:
//      most tokens are masked), coarser ones beyond -- one banned token at -1e9 or at the lowest float would otherwise put
//      the whole row into one bin -- and a bin for the smallest logit alone.  The bin is a monotone function of the
//      logit, so the bins are runs of the order, and integer masses make every sum exact.
//   3. cut_gather: every block redoes the scan of the histogram, which names the bin that holds the cut and what is still
//      to be covered inside it.  Tokens of earlier bins are certainly kept and take part in the draw at once; those of
//      the cut's bin (a few hundred at most over a row of logits) are collected in a list.
// sample_finish then finds the cut inside the list, lets the list's kept tokens take part, and emits token and
// log-probability.  With both cuts, the count is selected first (passes 2, 3 and cut_finish) and the mass among what it
// keeps.  Where a bin overflows the list (a crowd of thousands of tokens in a thousandth of the range, thousands of equal
// logits, or masked ones that the cut reaches) the finishing block goes over the row itself (row_cut).
// What bounds it: the passes' arithmetic per token (order keys, weights, LDS additions), then the finishing blocks, one per
// row.  A radix selection over the digits of the key took five passes, each with its own scan, and a draw over every
// entry.  Rows of 151936 entries, that selection -> these passes: 0.6 / 0.95 at 128 rows 217 -> 57 us, at one row 65 -> 26;
// top-k 50 198 -> 52 and 56 -> 28, also with masked tokens or logits rounded to 16 bits; a top-k cut among masked tokens
// 323 -> 87 and 58 -> 38; equal logits 360 -> 70 and 63 -> 23 (the cut follows from their number).  Slower at few rows is a
// crowd 30000 times narrower than the distance of an outlier above it (top-k: 197 -> 132 at 128 rows, 56 -> 76 at one):
// steps that follow such a crowd cost plain rows 5 % at 256 rows.
// ------------------------------------------------------------------------------------------------
constexpr int kCutBins = 1024;
constexpr int kCutList = 4096;
constexpr int kCutThreads = 512;
static_assert(kCutTile >= kSampleTile, "a slice has a partial of its own");

struct CutSel {            // after the scan of a histogram
  int32_t bin;             // the bin that holds the cut
  int32_t pad;
  unsigned long long rem;  // count or mass still to be covered inside it
};
struct CutRow {  // per row
  unsigned long long hist[2][kCutBins];  // selection 0: count (top-k), 1: mass (top-p)
  CutSel sel[2];
  uint32_t n_list[2];                    // tokens of the cut's bin, also where they are more than the list holds
  uint32_t lo[2], hi[2];                 // their smallest and largest key
  OrderCut cut_k;
  // per slice: largest and smallest key; the same of the finite logits (or 0, 0xffffffff); the largest minimum of two and
  // of four neighbouring logits, as keys
  uint32_t kmax[kCutSlices], kmin[kCutSlices], fmax[kCutSlices], fmin[kCutSlices], two[kCutSlices], four[kCutSlices];
  float unit_max[kCutUnits];             // +inf where a unit holds something that is not a number
  uint2 list[2][kCutList];               // (key, index)
};
static_assert(sizeof(CutRow) % 16 == 0, "rows lie one behind the other, histograms are read in pairs");

// Calls fn(i, z[i .. i + 3]) for the float4 groups [g_begin, g_end) of the row (V % 4 == 0, rows 16-byte aligned), kLoads
// 16-byte loads in flight per thread.
template <int kLoads, typename F>
__device__ __forceinline__ void for_each_group(const float* __restrict__ z, int g_begin, int g_end, int tid, int nthr, F fn) {
  for (int g0 = g_begin + tid; g0 < g_end; g0 += kLoads * nthr) {
    float4 v[kLoads];
#pragma unroll
    for (int e = 0; e < kLoads; ++e) {
      const int g = g0 + e * nthr;
      v[e] = g < g_end ? ((const float4*)z)[g] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int e = 0; e < kLoads; ++e) {
      const int g = g0 + e * nthr;
      if (g < g_end) fn(4 * g, v[e]);
    }
  }
}

__device__ __forceinline__ int signed_key(float z) {  // as a signed number in the order of order_key
  const int b = __float_as_int(z);
  return b ^ ((b >> 31) & 0x7fffffff);
}
__device__ __forceinline__ bool finite_bits(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

// units: of the slice, from its start; unit0: where the row keeps the first one's largest logit, or -1 (a row of more than
// kCutUnits, i.e. beyond 2^18 logits).
struct Slice { int g_begin, g_end, units, unit0; };
__device__ __forceinline__ Slice row_slice(int V) {
  const int n4 = V >> 2, per = cut_groups_per_slice(V, gridDim.x);
  const int g = min(n4, (int)blockIdx.x * per), g_end = min(n4, g + per);
  return Slice{g, g_end, (g_end - g + 63) >> 6, cut_keeps_units(V, gridDim.x) ? (int)blockIdx.x * cut_units_per_slice(V, gridDim.x) : -1};
}

// The row's largest logit, and the bins of a selection: of a mass, equal steps down from z_ref; of a count, 512 equal steps
// over r0, 256 over what follows up to r1, 254 over the rest, then one bin for the smallest logit.
struct CutBinning {
  float z_max, s_max;  // largest logit of the order; the same times 1/T
  float z_ref;         // where the bins begin
  float scale, scale1, scale2;  // bins per unit of the logit
  float r0, r1;
  uint32_t floor;      // bits of the row's smallest logit: masked tokens, mostly
  bool all;            // mass: no token has any (the largest score is not a finite number, or rounded by more than 22)
  bool equal;          // all logits are equal
  template <bool kMass>
  __device__ __forceinline__ int bin(float z) const {
    const float t = z_ref - z;
    if (kMass) return (int)fminf(t * scale, (float)(kCutBins - 1));  // of logits that have a mass
    if (t < r0) return (int)fmaxf(t * scale, 0.f);  // +inf as well; never the smallest logit
    if (__float_as_uint(z) == floor) return kCutBins - 1;
    if (!finite_bits(z)) return (int)__float_as_uint(z) < 0 ? kCutBins - 2 : 0;  // by its place in the order
    return (int)(t < r1 ? (t - r0) * scale1 + 512.f : fminf((t - r1) * scale2, 254.f) + 768.f);
  }
  // Leading tokens that are kept where that follows without a search (every token, or so many of the equal ones), or -1.
  template <bool kMass>
  __device__ __forceinline__ int prefix(int n_allowed, int V, float inv_t, unsigned long long target, unsigned long long p_fixed) const;
};
__device__ __forceinline__ CutBinning cut_binning(const CutRow& row, int n_slices, float inv_t, bool mass) {
  const int i = min((int)(threadIdx.x & (kCutSlices - 1)), n_slices - 1);  // both halves of a wave hold all slices
  uint32_t kmax = row.kmax[i], kmin = row.kmin[i], fmax = row.fmax[i], fmin = row.fmin[i], two = row.two[i], four = row.four[i];
  each_mask<kCutSlices / 2>([&](int o) __attribute__((always_inline)) {
    kmax = max(kmax, lane_xor(kmax, o));
    kmin = min(kmin, lane_xor(kmin, o));
    fmax = max(fmax, lane_xor(fmax, o));
    fmin = min(fmin, lane_xor(fmin, o));
    two = max(two, lane_xor(two, o));
    four = max(four, lane_xor(four, o));
  });
  CutBinning b;
  b.z_max = order_value(kmax);
  b.s_max = __fmul_rn(b.z_max, inv_t);
  b.all = mass && fexp_weight(__fmaf_rn(b.z_max, inv_t, -b.s_max)) == 0;
  b.z_ref = order_value(fmax);
  b.floor = __float_as_uint(order_value(kmin));
  b.equal = kmin == kmax;
  const auto steps = [](float n, float range) { const float q = n / range; return range > 0.f && finite_bits(q) ? q : 0.f; };
  const float range = b.z_ref - order_value(fmin);  // NaN without a finite logit
  b.r0 = b.r1 = b.scale1 = b.scale2 = 0.f;
  if (mass) {
    b.scale = steps(kCutBins - 1, fminf(range, 22.5f / inv_t));
  } else {
    const float d2 = b.z_ref - order_value(two), d4 = b.z_ref - order_value(four);
    const float bulk = d2 > 0.f ? fminf(4.f * d4, 64.f * d2) : 4.f * d4;
    b.r0 = bulk > 0.f ? fminf(range, bulk) : range;
    b.r1 = fminf(range, 32.f * b.r0);
    b.scale = steps(512.f, b.r0);
    b.scale1 = steps(256.f, b.r1 - b.r0);
    b.scale2 = steps(254.f, range - b.r1);
  }
  return b;
}

// One wave: the position (in scan order: descending or ascending bin) at which the running sum of `hist` first
// reaches `rem`; the last position is taken when none does.  Returns the bin; *rem_out = what is still to be covered
// inside it.  Every lane returns the same values.
// target(S): what is to be covered, given the sum of all bins.
template <bool kDescending, int kPer, typename F>
__device__ __forceinline__ int scan_select_n(const unsigned long long* hist, F target, int lane, unsigned long long* rem_out) {
  constexpr int n_bins = 64 * kPer;
  // this lane's kPer positions (consecutive in scan order), loaded once as 16-byte pairs
  unsigned long long c[kPer];
  const int first = kDescending ? n_bins - (lane + 1) * kPer : lane * kPer;  // lowest bin of the lane's range
#pragma unroll
  for (int e = 0; e < kPer; e += 2) {
    const ulonglong2 v = *(const ulonglong2*)(hist + first + e);
    c[kDescending ? kPer - 1 - e : e] = v.x;
    c[kDescending ? kPer - 2 - e : e + 1] = v.y;
  }
  unsigned long long local = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) local += c[e];
  unsigned long long incl = local;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const unsigned long long t = __shfl_up(incl, o, kWave);
    if (lane >= o) incl += t;
  }
  const unsigned long long rem = target(__shfl(incl, 63, kWave));
  unsigned long long cum = incl - local;  // sum of the positions before this lane's
  int hit = -1;
  unsigned long long before = 0;
#pragma unroll
  for (int e = 0; e < kPer; ++e) {
    const int pos = lane * kPer + e;
    if (hit < 0 && pos < n_bins - 1 && cum + c[e] >= rem) { hit = pos; before = cum; }
    if (pos < n_bins - 1) cum += c[e];  // in the last lane: ends as the sum of all positions but the last
  }
  const unsigned long long any = __ballot(hit >= 0);
  const int src = any ? (int)__builtin_ctzll(any) : 63;
  if (!any) { hit = n_bins - 1; before = cum; }
  hit = __shfl(hit, src, kWave);
  before = __shfl(before, src, kWave);
  *rem_out = rem - before;
  return kDescending ? n_bins - 1 - hit : hit;
}

// What a selection has to cover: max(1, floor(p_fixed * S / 2^32)) of the mass S of all allowed tokens, or `target`.
__device__ __forceinline__ unsigned long long mass_target(unsigned long long S, unsigned long long p_fixed) {
  const unsigned long long t = (__umul64hi(S, p_fixed) << 32) | ((S * p_fixed) >> 32);  // S < 2^50, p_fixed < 2^32
  return t < 1 ? 1 : t;
}

template <bool kMass>
__device__ __forceinline__ int CutBinning::prefix(int n_allowed, int V, float inv_t, unsigned long long target,
                                                  unsigned long long p_fixed) const {
  if (all) return V;
  if (!equal) return -1;
  if (!kMass) return (int)target;
  const unsigned long long w = fexp_weight(__fmaf_rn(z_max, inv_t, -s_max));  // not zero
  const unsigned long long n = (mass_target(w * (unsigned long long)n_allowed, p_fixed) + w - 1) / w;
  return (int)min(max(n, 1ull), (unsigned long long)n_allowed);  // scores beyond 10^9 may round to a weight that overflows
}

// grid (slices, rows): the slice's share of the row's range; clears the row's histograms and counters.
__global__ __launch_bounds__(kCutThreads) void cut_range_kernel(const float* __restrict__ logits, int V, CutRow* __restrict__ ws) {
  __shared__ uint32_t sh[6][kCutThreads / 64];
  const int r = blockIdx.y, tid = threadIdx.x;
  CutRow& row = ws[r];
  for (int i = blockIdx.x * kCutThreads + tid; i < 2 * kCutBins; i += gridDim.x * kCutThreads) (&row.hist[0][0])[i] = 0ull;
  if (blockIdx.x == 0 && tid < 2) { row.n_list[tid] = 0u; row.lo[tid] = 0xffffffffu; row.hi[tid] = 0u; }
  const Slice sl = row_slice(V);
  uint32_t kmax = 0, kmin = 0xffffffffu, fmax = 0, fmin = 0xffffffffu;
  int smax = (int)0x80000000, smin = 0x7fffffff;
  float two = -INFINITY, four = -INFINITY;
  const float4* z4 = (const float4*)(logits + (size_t)r * V);
  for (int g0 = sl.g_begin; g0 < sl.g_end; g0 += 4 * kCutThreads) {
    float4 v[4];
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int g = g0 + p * kCutThreads + tid;
      v[p] = z4[g < sl.g_end ? g : sl.g_end - 1];  // the last group again: changes nothing below
    }
    float tops[4];
    bool odd = false;
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const float sum = (v[p].x + v[p].y) + (v[p].z + v[p].w);  // not finite where one of them is not, or hardly ever besides
      odd |= !finite_bits(sum);
      tops[p] = sum != sum ? INFINITY : fmaxf(fmaxf(v[p].x, v[p].y), fmaxf(v[p].z, v[p].w));
      const float a = fminf(v[p].x, v[p].y), b = fminf(v[p].z, v[p].w);
      two = fmaxf(two, fmaxf(a, b));
      four = fmaxf(four, fminf(a, b));
      if (!finite_bits(sum)) continue;
      const int k0 = signed_key(v[p].x), k1 = signed_key(v[p].y), k2 = signed_key(v[p].z), k3 = signed_key(v[p].w);
      smax = max(smax, max(max(k0, k1), max(k2, k3)));
      smin = min(smin, min(min(k0, k1), min(k2, k3)));
    }
    if (odd) {
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        const float zs[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const uint32_t k = order_key(zs[e]);
          kmax = max(kmax, k);
          kmin = min(kmin, k);
          fmax = max(fmax, finite_bits(zs[e]) ? k : 0u);
          fmin = min(fmin, finite_bits(zs[e]) ? k : 0xffffffffu);
        }
      }
    }
    // the four units' maxima at once, that of load p in lane p: every step halves the values a lane carries
    const bool up1 = tid & 1, up2 = tid & 2;
    const float t0 = fmaxf(up1 ? tops[1] : tops[0], lane_xor(up1 ? tops[0] : tops[1], 1));
    const float t1 = fmaxf(up1 ? tops[3] : tops[2], lane_xor(up1 ? tops[2] : tops[3], 1));
    float top = fmaxf(up2 ? t1 : t0, lane_xor(up2 ? t0 : t1, 2));
    top = lane_max(lane_max(lane_max(lane_max(top, 4), 8), 16), 32);
    const int unit = ((g0 - sl.g_begin) >> 6) + (tid & 63) * (kCutThreads / 64) + (tid >> 6);
    if (sl.unit0 >= 0 && (tid & 63) < 4 && unit < sl.units) row.unit_max[sl.unit0 + unit] = top;
  }
  if (smax >= smin) {  // of groups without anything odd: order_key is the signed key with its sign turned
    kmax = max(kmax, (uint32_t)smax ^ 0x80000000u);
    kmin = min(kmin, (uint32_t)smin ^ 0x80000000u);
    fmax = max(fmax, (uint32_t)smax ^ 0x80000000u);
    fmin = min(fmin, (uint32_t)smin ^ 0x80000000u);
  }
  uint32_t ktwo = order_key(two), kfour = order_key(four);
  each_mask([&](int o) __attribute__((always_inline)) {
    kmax = max(kmax, lane_xor(kmax, o));
    kmin = min(kmin, lane_xor(kmin, o));
    fmax = max(fmax, lane_xor(fmax, o));
    fmin = min(fmin, lane_xor(fmin, o));
    ktwo = max(ktwo, lane_xor(ktwo, o));
    kfour = max(kfour, lane_xor(kfour, o));
  });
  if ((tid & 63) == 0) { sh[0][tid >> 6] = kmax; sh[1][tid >> 6] = fmax; sh[2][tid >> 6] = fmin; sh[3][tid >> 6] = kfour; sh[4][tid >> 6] = kmin; sh[5][tid >> 6] = ktwo; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kCutThreads / 64; ++w) {
      kmax = max(kmax, sh[0][w]);
      fmax = max(fmax, sh[1][w]);
      fmin = min(fmin, sh[2][w]);
      kfour = max(kfour, sh[3][w]);
      kmin = min(kmin, sh[4][w]);
      ktwo = max(ktwo, sh[5][w]);
    }
    row.kmax[blockIdx.x] = kmax;
    row.kmin[blockIdx.x] = kmin;
    row.fmax[blockIdx.x] = fmax;
    row.fmin[blockIdx.x] = fmin;
    row.two[blockIdx.x] = ktwo;
    row.four[blockIdx.x] = kfour;
  }
}

// h[bin[e]] += w[e], and with kCount n[bin[e]] += 1, for four tokens per lane; bin < 0: none.  Where all lanes' tokens go
// to one bin (equal logits, or a crowd in one bin) they are added up first: a hundred thousand additions to one LDS word
// would take longer than everything else.
template <bool kCount>
__device__ __forceinline__ void add_to_bins(unsigned long long* h, uint32_t* n, const int (&bin)[4], const unsigned long long (&w)[4]) {
  if (bin[0] == bin[1] && bin[0] == bin[2] && bin[0] == bin[3]) {
    if (bin[0] < 0) return;
    unsigned long long sum = (w[0] + w[1]) + (w[2] + w[3]);
    const int first = __builtin_amdgcn_readfirstlane(bin[0]);
    if (__ballot(bin[0] == first) == ~0ull) {  // every lane of the wave
      each_mask([&](int o) __attribute__((always_inline)) { sum += lane_xor(sum, o); });
      if ((threadIdx.x & 63) == 0) {
        atomicAdd(&h[first], sum);
        if (kCount) atomicAdd(&n[first], 256u);
      }
    } else {
      atomicAdd(&h[bin[0]], sum);
      if (kCount) atomicAdd(&n[bin[0]], 4u);
    }
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (bin[e] >= 0) {
      atomicAdd(&h[bin[e]], w[e]);
      if (kCount) atomicAdd(&n[bin[e]], 1u);
    }
}

// grid (slices, rows): the slice's share of the histogram of selection kMass, among the tokens that `use_k`'s cut keeps.
template <bool kMass>
__global__ __launch_bounds__(kCutThreads) void cut_hist_kernel(const float* __restrict__ logits, int V, float inv_t, int use_k,
                                                               CutRow* __restrict__ ws) {
  __shared__ __align__(16) unsigned long long lh[kCutBins];
  const int r = blockIdx.y, tid = threadIdx.x;
  CutRow& row = ws[r];
  const CutBinning cb = cut_binning(row, gridDim.x, inv_t, kMass);
  if (cb.all || cb.equal) return;  // block-uniform: no search
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  for (int b = tid; b < kCutBins; b += kCutThreads) lh[b] = 0ull;
  __syncthreads();
  const Slice sl = row_slice(V);
  const auto scan = [&](auto near_c, auto all_c) __attribute__((always_inline)) {
    for_each_group<4>(logits + (size_t)r * V, sl.g_begin, sl.g_end, tid, kCutThreads, [&](int i0, float4 v) {
      const float zs[4] = {v.x, v.y, v.z, v.w};
      if constexpr (kMass) {
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float x = __fmaf_rn(zs[e], inv_t, -cb.s_max);
          if (!(x > -22.0f)) continue;  // weight zero
          if (!decltype(all_c)::value && use_k && !kept_by(allowed, order_key(zs[e]), i0 + e)) continue;
          atomicAdd(&lh[cb.bin<true>(zs[e])], fexp_weight<decltype(near_c)::value>(x));
        }
      } else {
        int bins[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          bins[e] = cb.bin<false>(zs[e]);
          if (bins[e] == kCutBins - 1) bins[e] = -1;  // a scan that does not reach its count before the last bin ends there
        }
        const unsigned long long w[4] = {1, 1, 1, 1};
        add_to_bins<false>(lh, nullptr, bins, w);
      }
    });
  };
  // The scan is bound by its instructions (45 per token): the usual row does without the branch for weights beyond one and
  // without a cut before this one, 20.4 -> 18 us at 128 rows (16.3 in the present slices).  Largest scores below 2^20 are off by less than a sixteenth
  // when rounded: no score exceeds them by more.
  if (!kMass || (fabsf(cb.s_max) <= 0x1p20f && !use_k)) scan(std::true_type{}, std::true_type{});  // block-uniform
  else scan(std::false_type{}, std::false_type{});
  __syncthreads();
  for (int b = tid; b < kCutBins; b += kCutThreads)
    if (lh[b] != 0ull) atomicAdd(&row.hist[kMass][b], lh[b]);
}

// What one block knows of a draw: best score, and the sum of exp((z - z_max) / T) in whole units of 2^-40.  Neither
// depends on the order or the grouping in which tokens are added (a list's order changes from run to run, the slices
// with the number of rows): a row's log-probability has the same bits in every call and in every batch.  The units are
// finer than an fp32 sum resolves: at most 2^-41 lost per token, and a sum below 2^62 for vocabularies below 2^22.
// Against 64 bits the log-probabilities are off by 4e-8 (relative) where an fp32 log-sum-exp of the scores was off by
// 2.8e-7; 128 rows of 151936 entries at 0.6 / 0.95: 75.1 -> 73.7 us.  A kept logit that is not a number is never drawn
// and makes the log-probability not a number.
struct Draw {
  Best best;
  unsigned long long sum;
  static constexpr unsigned long long kNan = 1ull << 63;  // stays set through every addition
  __device__ __forceinline__ static unsigned long long plus(unsigned long long a, unsigned long long b) {
    return ((a + b) & ~kNan) | ((a | b) & kNan);
  }
  __device__ __forceinline__ void add(int i, float z, float z_max, float inv_t, uint32_t rnd) {
    const float y = __fmaf_rn(z, inv_t, gumbel(rnd));
    if (y == y) best = better(best, Best{y, i, z});
    const float e = __expf(__fmul_rn(__fsub_rn(z, z_max), inv_t));  // at most 1
    sum = plus(sum, e == e ? (unsigned long long)__fmaf_rn(e, 0x1p40f, 0.5f) : kNan);
  }
  __device__ __forceinline__ void merge(const Draw& o) {
    best = better(best, o.best);
    sum = plus(sum, o.sum);
  }
  __device__ __forceinline__ float logprob(float z, float z_max, float inv_t) const {
    return sum & kNan ? __uint_as_float(0x7fc00000u) : __fmul_rn(__fsub_rn(z, z_max), inv_t) - logf((float)sum * 0x1p-40f);
  }
};
// The random word of token i.
__device__ __forceinline__ uint32_t token_bits(uint32_t i, uint32_t pos, uint32_t seq, uint32_t seed_lo, uint32_t seed_hi) {
  uint32_t rnd[4];
  philox4x32_10(i >> 2, pos, seq, 0u, seed_lo, seed_hi, rnd);
  return (i & 2) ? ((i & 1) ? rnd[3] : rnd[2]) : ((i & 1) ? rnd[1] : rnd[0]);
}
__device__ __forceinline__ Draw empty_draw() { return Draw{Best{-INFINITY, -1, 0.f}, 0ull}; }
// The block's draw, in thread 0.
template <int kThreads>
__device__ __forceinline__ Draw block_draw(Draw d, Draw (&sh)[kThreads / 64]) {
  each_mask([&](int o) __attribute__((always_inline)) {
    d.best = best_of_lanes(d.best, o);
    d.sum = Draw::plus(d.sum, lane_xor(d.sum, o));
  });
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = d;
  __syncthreads();
  if (threadIdx.x == 0)
    for (int w = 1; w < kThreads / 64; ++w) d.merge(sh[w]);
  return d;
}

struct DrawArgs {
  const RowMeta* rows;
  int pos_offset;
  uint32_t seed_lo, seed_hi;
  const int32_t* forced;
  float* forced_z;
  float* part;  // [rows][gridDim.x][kSamplePartFloats]
};

// grid (slices, rows): names the cut's bin, lists the slice's tokens in it and (kDraw) draws among the slice's tokens of
// earlier bins.
template <bool kMass, bool kDraw>
__global__ __launch_bounds__(kCutThreads) void cut_gather_kernel(const float* __restrict__ logits, int V, float inv_t, int use_k,
                                                                 unsigned long long target, unsigned long long p_fixed,
                                                                 CutRow* __restrict__ ws, DrawArgs da) {
  __shared__ CutSel sh_sel;
  __shared__ Draw sh_draw[kCutThreads / 64];
  constexpr int kKept = kDraw ? 2048 : 1;  // certainly kept tokens, drawn among after the scan with all lanes busy
  __shared__ uint2 sh_list[kCutList], sh_kept[kKept];
  __shared__ uint32_t sh_n, sh_at, sh_nk, sh_lo, sh_hi;
  const int r = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  CutRow& row = ws[r];
  const Slice sl = row_slice(V);
  uint32_t pos = 0, seq = 0;
  int f = -1;
  if (kDraw) {
    const RowMeta rm = da.rows[r];
    pos = (uint32_t)(rm.pos + da.pos_offset);
    seq = (uint32_t)rm.seq;
    if (da.forced) f = da.forced[r];
    // cut off, i.e. of probability zero, unless it is found among the kept tokens, here or by sample_finish
    if (tid == 0 && f >= 4 * sl.g_begin && f < 4 * sl.g_end) da.forced_z[r] = -INFINITY;
  }
  const CutBinning cb = cut_binning(row, gridDim.x, inv_t, kMass);
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  if (tid < 64) {
    const unsigned long long* h = row.hist[kMass];
    CutSel sel{0, 0, 0ull};
    sel.bin = scan_select_n<false, kCutBins / 64>(h, [&](unsigned long long S) { return kMass ? mass_target(S, p_fixed) : target; }, tid, &sel.rem);
    if (tid == 0) {
      sh_sel = sel;
      sh_n = sh_nk = sh_hi = 0u;
      sh_lo = 0xffffffffu;
      if (blockIdx.x == 0) row.sel[kMass] = sel;
    }
  }
  __syncthreads();
  const int cut_bin = sh_sel.bin;
  const float* z = logits + (size_t)r * V;
  Draw d = empty_draw();
  auto draw_token = [&](int i, float zi) {
    d.add(i, zi, cb.z_max, inv_t, token_bits((uint32_t)i, pos, seq, da.seed_lo, da.seed_hi));
  };
  // block-uniform
  const int n_prefix = cb.prefix<kMass>(use_k ? allowed.idx + 1 : V, V, inv_t, target, p_fixed);
  if (n_prefix >= 0 && !kDraw) {
    if (blockIdx.x == 0 && tid == 0) row.cut_k = OrderCut{order_key(cb.z_max), n_prefix - 1};
    return;
  }
  if (n_prefix >= 0) {
    for_each_group<4>(z, sl.g_begin, sl.g_end, tid, kCutThreads, [&](int i0, float4 v) {
      const float zs[4] = {v.x, v.y, v.z, v.w};
      uint32_t rnd[4];
      philox4x32_10((uint32_t)i0 >> 2, pos, seq, 0u, da.seed_lo, da.seed_hi, rnd);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool kept = i0 + e < n_prefix;
        if (kept) d.add(i0 + e, zs[e], cb.z_max, inv_t, rnd[e]);
        if (kept && f == i0 + e) da.forced_z[r] = zs[e];
      }
    });
  } else {
    uint32_t lo = 0xffffffffu, hi = 0u;
    // one token of the cut's bin or an earlier one
    const auto token = [&](int i, float zi) __attribute__((always_inline)) {
      const uint32_t k = order_key(zi);
      if (use_k && !kept_by(allowed, k, i)) return;
      if (cb.bin<kMass>(zi) == cut_bin) {
        if (kMass && !(__fmaf_rn(zi, inv_t, -cb.s_max) > -22.0f)) return;  // weight zero: never the cut, always behind it
        const uint32_t at = atomicAdd(&sh_n, 1u);
        if (at < (uint32_t)kCutList) sh_list[at] = make_uint2(k, (uint32_t)i);
        lo = min(lo, k);
        hi = max(hi, k);
      } else if (kDraw) {
        const uint32_t at = atomicAdd(&sh_nk, 1u);
        if (at < (uint32_t)kKept) sh_kept[at] = make_uint2(__float_as_uint(zi), (uint32_t)i);
        else draw_token(i, zi);
        if (f == i) da.forced_z[r] = zi;
      }
    };
    // A wave takes every eighth unit, and of those only the ones whose largest logit is in the cut's bin or before it (the
    // bin is a monotone function of the logit): where some dozens of tokens are kept, most of the row is not read again.
    // The code for a token exists once: sixteen copies of it, drawing included, were fetched past cold by every block.
    // 128 rows of 151936 entries, 0.6 / 0.95 (100 kept): this kernel 25.9 -> 14.9 us (14.1 in the present slices); 1.0 / 0.95
    // (14000 kept) all 113 -> 84.
    const bool read_all = sl.unit0 < 0 || sl.units <= 4 * (kCutThreads / 64);  // all at once is faster than asking first
    for (int u0 = wave; u0 < sl.units; u0 += 64 * (kCutThreads / 64)) {
      const int u = u0 + lane * (kCutThreads / 64);
      const bool there = u < sl.units;
      const float most = read_all ? INFINITY : row.unit_max[sl.unit0 + (there ? u : 0)];
      unsigned long long left = __ballot(there && (most == INFINITY || cb.bin<kMass>(most) <= cut_bin));
      while (left) {
        float4 v[4];
        int g[4];
        const int n_units = min(4, __popcll(left));  // wave-uniform
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          g[p] = left ? sl.g_begin + 64 * (u0 + (int)__builtin_ctzll(left) * (kCutThreads / 64)) + lane : sl.g_end;
          left &= left - 1;
          v[p] = ((const float4*)z)[min(g[p], sl.g_end - 1)];
        }
        uint32_t mask = 0;  // of the thread's sixteen tokens
#pragma unroll
        for (int p = 0; p < 4; ++p) {
          // most groups lie behind the cut's bin as a whole; fmaxf skips a NaN, which the sum shows
          const float top = fmaxf(fmaxf(v[p].x, v[p].y), fmaxf(v[p].z, v[p].w)), sum = (v[p].x + v[p].y) + (v[p].z + v[p].w);
          if (g[p] >= sl.g_end || (cb.bin<kMass>(top) > cut_bin && (kMass || sum == sum))) continue;
          const float zs[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
          for (int e = 0; e < 4; ++e) mask |= cb.bin<kMass>(zs[e]) <= cut_bin ? 1u << (4 * p + e) : 0u;
        }
        // A count that ends among thousands of equal or nearly equal logits finds whole units in the cut's bin: their tokens
        // take their places at once.  128 rows of 151936 entries, one by one -> at once, this kernel: ten tokens above equal
        // ones 54 -> 40 us, one token above a crowd 51 -> 37.
        if constexpr (!kMass) {
          if (__ballot(mask == (1u << 4 * n_units) - 1u) == ~0ull) {
            uint32_t k_lo = 0xffffffffu, k_hi = 0u;
            bool in_bin = true;
#pragma unroll
            for (int p = 0; p < 4; ++p) {
              if (p >= n_units) continue;
              const float zs[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
              for (int e = 0; e < 4; ++e) {
                in_bin &= cb.bin<kMass>(zs[e]) == cut_bin;
                k_lo = min(k_lo, order_key(zs[e]));
                k_hi = max(k_hi, order_key(zs[e]));
              }
            }
            if (__ballot(in_bin) == ~0ull) {
              uint32_t at = 0;
              if (lane == 0) at = atomicAdd(&sh_n, 256u * n_units);
              at = __builtin_amdgcn_readfirstlane(at) + lane;
#pragma unroll
              for (int p = 0; p < 4; ++p) {
                if (p >= n_units) continue;
                const float zs[4] = {v[p].x, v[p].y, v[p].z, v[p].w};
#pragma unroll
                for (int e = 0; e < 4; ++e, at += 64)
                  if (at < (uint32_t)kCutList) sh_list[at] = make_uint2(order_key(zs[e]), (uint32_t)(4 * g[p] + e));
              }
              lo = min(lo, k_lo);
              hi = max(hi, k_hi);
              mask = 0;
            }
          }
        }
        while (mask) {
          const int at = __builtin_ctz(mask), p = at >> 2, e = at & 3;
          mask &= mask - 1;
          const float4 a = p & 1 ? v[1] : v[0], b = p & 1 ? v[3] : v[2], c = p & 2 ? b : a;
          const int ga = p & 1 ? g[1] : g[0], gb = p & 1 ? g[3] : g[2];
          token(4 * (p & 2 ? gb : ga) + e, e & 2 ? (e & 1 ? c.w : c.z) : (e & 1 ? c.y : c.x));
        }
      }
    }
    if (lo <= hi) { atomicMin(&sh_lo, lo); atomicMax(&sh_hi, hi); }
    __syncthreads();
    const uint32_t n_own = sh_n;
    if (tid == 0 && n_own > 0) {
      sh_at = atomicAdd(&row.n_list[kMass], n_own);
      atomicMin(&row.lo[kMass], sh_lo);
      atomicMax(&row.hi[kMass], sh_hi);
    }
    __syncthreads();
    if (n_own > 0)
      for (uint32_t t = tid; t < min(n_own, (uint32_t)kCutList) && sh_at + t < (uint32_t)kCutList; t += kCutThreads) row.list[kMass][sh_at + t] = sh_list[t];
    if (kDraw)
      for (uint32_t t = tid; t < min(sh_nk, (uint32_t)kKept); t += kCutThreads) draw_token((int)sh_kept[t].y, __uint_as_float(sh_kept[t].x));
  }
  if (!kDraw) return;
  d = block_draw<kCutThreads>(d, sh_draw);
  if (tid == 0) {
    float* p = da.part + ((size_t)r * gridDim.x + blockIdx.x) * kSamplePartFloats;
    *(float4*)p = make_float4(d.best.y, __int_as_float(d.best.idx), d.best.z, 0.f);
    *(unsigned long long*)(p + 4) = d.sum;
  }
}

// A token's place in the order as one number, descending: its key and, below it, its index from the end.
constexpr int kIndexBits = 22;  // vocabularies are below 2^22
constexpr uint32_t kIndexMask = (1u << kIndexBits) - 1;
typedef unsigned long long place_t;
__device__ __forceinline__ place_t place_of(uint32_t key, uint32_t i) { return ((place_t)key << kIndexBits) | (kIndexMask - i); }
__device__ __forceinline__ OrderCut cut_at(place_t c) { return OrderCut{(uint32_t)(c >> kIndexBits), (int32_t)(kIndexMask - ((uint32_t)c & kIndexMask))}; }

constexpr int kFinishThreads = 1024;
constexpr int kFinishWaves = kFinishThreads / 64;
constexpr int kCutFew = 512;
struct FinishLds {
  __align__(16) unsigned long long hist[kCutBins];
  place_t few[kCutFew];
  unsigned long long few_weight[kCutFew];
  uint32_t count[kCutBins];
  uint2 list[kCutList];
  Draw draw[kFinishWaves];
  place_t cut;
  uint32_t n;
  uint32_t found[2][4][kFinishWaves];
};
static_assert(kCutFew <= kFinishThreads, "one thread each");

template <bool kMass>
__device__ __forceinline__ unsigned long long token_weight(uint32_t key, float inv_t, float s_max) {
  return kMass ? fexp_weight(__fmaf_rn(order_value(key), inv_t, -s_max)) : 1ull;
}

// The cut among the n tokens of sh.list that lie in places lo .. hi, of whose count or mass `rem` is to be covered, in
// every thread: equal steps of the place until a step holds few tokens (one round, unless more than kCutFew have the
// same key), then those against each other.
template <bool kMass>
__device__ place_t list_cut(int n, place_t lo, place_t hi, unsigned long long rem, float inv_t, float s_max, FinishLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63;
  int n_few;
  do {
    const int shift = max(0, 54 - (int)__clzll((long long)(hi - lo)));  // (hi - lo) >> shift < kCutBins
    __syncthreads();
    for (int b = tid; b < kCutBins; b += kFinishThreads) sh.hist[b] = 0ull;
    if (tid == 0) sh.n = 0u;
    __syncthreads();
    for (int t = tid; t < n; t += kFinishThreads) {
      const uint2 e = sh.list[t];
      const place_t c = place_of(e.x, e.y);
      if (c >= lo && c <= hi) atomicAdd(&sh.hist[(hi - c) >> shift], token_weight<kMass>(e.x, inv_t, s_max));
    }
    __syncthreads();
    unsigned long long left;  // the same in every wave
    const int step = scan_select_n<false, kCutBins / 64>(sh.hist, [&](unsigned long long) { return rem; }, lane, &left);
    rem = left;
    hi -= min((place_t)step << shift, hi - lo);
    lo = max(lo, hi - min(hi, ((place_t)1 << shift) - 1));
    for (int t = tid; t < n; t += kFinishThreads) {
      const uint2 e = sh.list[t];
      const place_t c = place_of(e.x, e.y);
      if (c < lo || c > hi) continue;
      const uint32_t at = atomicAdd(&sh.n, 1u);
      if (at < (uint32_t)kCutFew) { sh.few[at] = c; sh.few_weight[at] = token_weight<kMass>(e.x, inv_t, s_max); }
    }
    __syncthreads();
    n_few = (int)sh.n;
  } while (n_few > kCutFew);  // a range shrinks to a 512th at least in every round, to a single place at last
  if (tid == 0) sh.cut = lo;
  __syncthreads();
  if (tid < n_few) {
    const place_t c = sh.few[tid];
    unsigned long long before = 0;
    for (int u = 0; u < n_few; ++u)
      if (sh.few[u] > c) before += sh.few_weight[u];
    if (before < rem && rem <= before + sh.few_weight[tid]) atomicMax(&sh.cut, c);  // one token
  }
  __syncthreads();
  return sh.cut;
}

// The `need`-th token with this key (in the order of the index), found chunk by chunk from the row's start; in every
// thread.  Where the row has fewer, the last index.
__device__ place_t nth_of_key(const float* __restrict__ z, int V, uint32_t key, unsigned long long need, FinishLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, n4 = V >> 2;
  unsigned long long seen = 0;
  if (tid == 0) sh.cut = place_of(key, kIndexMask);
  int turn = 0;
  for (int g0 = 0; g0 < n4; g0 += 4 * kFinishThreads, turn ^= 1) {  // the buffers in turn: one barrier per chunk
    unsigned long long m[4][4];  // lanes whose element e of part p has the key
#pragma unroll
    for (int p = 0; p < 4; ++p) {
      const int g = g0 + p * kFinishThreads + tid;
      const float4 v = g < n4 ? ((const float4*)z)[g] : make_float4(0.f, 0.f, 0.f, 0.f);
      m[p][0] = __ballot(g < n4 && order_key(v.x) == key);
      m[p][1] = __ballot(g < n4 && order_key(v.y) == key);
      m[p][2] = __ballot(g < n4 && order_key(v.z) == key);
      m[p][3] = __ballot(g < n4 && order_key(v.w) == key);
      if (lane == 0)
        sh.found[turn][p][wave] = __builtin_popcountll(m[p][0]) + __builtin_popcountll(m[p][1]) + __builtin_popcountll(m[p][2]) + __builtin_popcountll(m[p][3]);
    }
    __syncthreads();
    unsigned long long before = seen, mine[4];
#pragma unroll
    for (int p = 0; p < 4; ++p)
      for (int w = 0; w < kFinishWaves; ++w) {
        if (w == wave) mine[p] = before;
        before += sh.found[turn][p][w];
      }
    if (before >= need) {  // block-uniform: it is in this chunk
      const unsigned long long below = (1ull << lane) - 1;
#pragma unroll
      for (int p = 0; p < 4; ++p) {
        unsigned long long at = mine[p];
#pragma unroll
        for (int e = 0; e < 4; ++e) at += __builtin_popcountll(m[p][e] & below);
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (m[p][e] >> lane & 1ull) {
            if (++at == need) sh.cut = place_of(key, 4u * (uint32_t)(g0 + p * kFinishThreads + tid) + e);
          }
      }
      break;
    }
    seen = before;
  }
  __syncthreads();
  return sh.cut;
}

// The row's cut of selection kMass, in every thread.  The list of its bin, as far as the cut depends on it, is in sh.list
// (*n_list tokens) afterwards; kept(i0, mask, z) is called for groups of four tokens of the bin of which those in the mask
// are kept without being in the list.
// A bin with more tokens than a list holds is narrowed first: 1024 steps of the key at a time, each a pass over the row,
// until a list holds a step's tokens (one pass, hardly ever two), or all have one key, of which the index then decides.
template <bool kMass, typename F>
__device__ place_t row_cut(const float* __restrict__ z, int V, float inv_t, const CutBinning& cb, const CutRow& row, int use_k,
                           FinishLds& sh, int* n_list, F kept) {
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t n = row.n_list[kMass], lo = row.lo[kMass], hi = row.hi[kMass];
  unsigned long long rem = row.sel[kMass].rem;
  if (n <= (uint32_t)kCutList) {
    for (int t = tid; t < (int)n; t += kFinishThreads) sh.list[t] = row.list[kMass][t];
    *n_list = (int)n;
    return list_cut<kMass>((int)n, (place_t)lo << kIndexBits, place_of(hi, 0u), rem, inv_t, cb.s_max, sh);
  }
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  const uint32_t top = hi;
  while (n > (uint32_t)kCutList && lo < hi) {
    const int shift = max(0, 22 - (int)__clz((int)(hi - lo)));  // (hi - lo) >> shift < kCutBins
    __syncthreads();
    for (int b = tid; b < kCutBins; b += kFinishThreads) { sh.hist[b] = 0ull; sh.count[b] = 0u; }
    __syncthreads();
    for_each_group<4>(z, 0, V >> 2, tid, kFinishThreads, [&](int i0, float4 v) {
      const float zs[4] = {v.x, v.y, v.z, v.w};
      int bins[4];
      unsigned long long w[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t k = order_key(zs[e]);
        const bool use = hi - k <= hi - lo && (!use_k || kept_by(allowed, k, i0 + e));
        bins[e] = use ? (int)((hi - k) >> shift) : -1;
        w[e] = !kMass ? 1ull : use ? token_weight<kMass>(k, inv_t, cb.s_max) : 0ull;
      }
      add_to_bins<kMass>(sh.hist, sh.count, bins, w);
    });
    __syncthreads();
    unsigned long long left;  // the same in every wave
    const int step = scan_select_n<false, kCutBins / 64>(sh.hist, [&](unsigned long long) { return rem; }, lane, &left);
    n = kMass ? sh.count[step] : (uint32_t)sh.hist[step];
    rem = left;
    hi -= min((uint32_t)step << shift, hi - lo);
    lo = max(lo, hi - min(hi, (1u << shift) - 1));
  }
  __syncthreads();
  place_t cut = (place_t)lo << kIndexBits;
  int g_end = V >> 2;
  const bool listed = n <= (uint32_t)kCutList;  // block-uniform
  if (!listed) {
    unsigned long long need = rem;
    if (kMass) {
      const unsigned long long w = token_weight<kMass>(lo, inv_t, cb.s_max);
      need = w > 0 ? max((rem + w - 1) / w, 1ull) : 1ull;
    }
    cut = nth_of_key(z, V, lo, need, sh);
    if (top == lo) g_end = min(g_end, cut_at(cut).idx / 4 + 1);  // nothing behind it
  }
  if (tid == 0) sh.n = 0u;
  __syncthreads();
  for_each_group<4>(z, 0, g_end, tid, kFinishThreads, [&](int i0, float4 v) {
    const float zs[4] = {v.x, v.y, v.z, v.w};
    uint32_t mask = 0;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const uint32_t k = order_key(zs[e]);
      if (k < lo || k > top) continue;
      if (k > hi || (!listed && place_of(k, (uint32_t)(i0 + e)) >= cut)) {
        mask |= 1u << e;
      } else if (listed && (!use_k || kept_by(allowed, k, i0 + e))) {
        const uint32_t at = atomicAdd(&sh.n, 1u);
        if (at < (uint32_t)kCutList) sh.list[at] = make_uint2(k, (uint32_t)(i0 + e));
      }
    }
    if (mask) kept(i0, mask, zs);
  });
  __syncthreads();
  *n_list = min((int)sh.n, kCutList);
  return listed ? list_cut<kMass>(*n_list, (place_t)lo << kIndexBits, place_of(hi, 0u), rem, inv_t, cb.s_max, sh) : cut;
}

// grid (rows): the top-k cut of a row that a top-p cut will follow.
__global__ __launch_bounds__(kFinishThreads) void cut_finish_kernel(const float* __restrict__ logits, int V, float inv_t, int n_slices,
                                                                    CutRow* __restrict__ ws) {
  __shared__ FinishLds sh;
  CutRow& row = ws[blockIdx.x];
  const CutBinning cb = cut_binning(row, n_slices, inv_t, false);
  if (cb.equal) return;  // cut_gather wrote the cut
  int n;
  const place_t cut = row_cut<false>(logits + (size_t)blockIdx.x * V, V, inv_t, cb, row, 0, sh, &n,
                                     [](int, uint32_t, const float*) {});
  if (threadIdx.x == 0) row.cut_k = cut_at(cut);
}

// grid (rows): the final cut, the draw among the tokens of its bin, and the result.
template <bool kMass>
__global__ __launch_bounds__(kFinishThreads) void sample_finish_kernel(const float* __restrict__ logits, int V, float inv_t,
                                                                       int n_slices, int use_k, const CutRow* __restrict__ ws,
                                                                       DrawArgs da, int32_t* __restrict__ out_tok,
                                                                       float* __restrict__ out_lp, int32_t* __restrict__ last_tok) {
  __shared__ FinishLds sh;
  const int r = blockIdx.x, tid = threadIdx.x;
  const CutRow& row = ws[r];
  const float* z = logits + (size_t)r * V;
  const CutBinning cb = cut_binning(row, n_slices, inv_t, kMass);
  const RowMeta rm = da.rows[r];
  const uint32_t pos = (uint32_t)(rm.pos + da.pos_offset), seq = (uint32_t)rm.seq;
  const int f = da.forced ? da.forced[r] : -1;
  __shared__ float sh_fz;
  Draw d = empty_draw();
  if (tid == 0 && f >= 0 && f < V) sh_fz = da.forced_z[r];
  if (!cb.all && !cb.equal) {  // block-uniform
    int n;
    const place_t cut = row_cut<kMass>(z, V, inv_t, cb, row, use_k, sh, &n, [&](int i0, uint32_t before, const float (&zs)[4]) {
      uint32_t rnd[4];
      philox4x32_10((uint32_t)i0 >> 2, pos, seq, 0u, da.seed_lo, da.seed_hi, rnd);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (before >> e & 1u) {
          d.add(i0 + e, zs[e], cb.z_max, inv_t, rnd[e]);
          if (i0 + e == f) sh_fz = zs[e];
        }
    });
    for (int t = tid; t < n; t += kFinishThreads) {
      const uint2 e = sh.list[t];
      if (place_of(e.x, e.y) < cut) continue;
      const float zi = order_value(e.x);
      d.add((int)e.y, zi, cb.z_max, inv_t, token_bits(e.y, pos, seq, da.seed_lo, da.seed_hi));
      if ((int)e.y == f) sh_fz = zi;
    }
  }
  for (int t = tid; t < n_slices; t += kFinishThreads) {
    const float* p = da.part + ((size_t)r * n_slices + t) * kSamplePartFloats;
    d.merge(Draw{Best{p[0], __float_as_int(p[1]), p[2]}, *(const unsigned long long*)(p + 4)});
  }
  d = block_draw<kFinishThreads>(d, sh.draw);  // its barrier also publishes sh_fz
  if (tid == 0) {
    int tok = d.best.idx < 0 ? 0 : d.best.idx;  // idx < 0 only when every score was NaN
    float zt = d.best.z;
    if (f >= 0 && f < V) { tok = f; zt = sh_fz; }
    out_tok[r] = tok;
    if (last_tok != nullptr) last_tok[rm.seq] = tok;
    out_lp[r] = d.logprob(zt, cb.z_max, inv_t);
  }
}

}  // namespace

size_t sample_cut_bytes_per_row() { return sizeof(CutRow); }

namespace {

// Truncated sampling of M rows (inv_t = 1/T > 0).  part holds at least ceil(V / kSampleTile) partials per row.
void launch_sample_cut(hipStream_t st, const float* logits, int M, int V, float inv_t, int top_k, float top_p, const DrawArgs& da,
                       CutRow* ws, int32_t* out_tokens, float* out_logprobs, int32_t* last_tok) {
  const bool use_k = top_k > 0 && top_k < V, use_p = top_p > 0.0f && top_p < 1.0f;
  const unsigned long long K = (unsigned long long)top_k, P = (unsigned long long)(top_p * 4294967296.0f);  // exact scaling, truncated
  const int slices = cut_slices(M, V);
  const dim3 grid(slices, M);
  cut_range_kernel<<<grid, kCutThreads, 0, st>>>(logits, V, ws);
  if (use_k) {
    cut_hist_kernel<false><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, ws);
    if (!use_p) {
      cut_gather_kernel<false, true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, K, 0ull, ws, da);
      sample_finish_kernel<false><<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, 0, ws, da, out_tokens, out_logprobs, last_tok);
      return;
    }
    cut_gather_kernel<false, false><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, K, 0ull, ws, da);
    cut_finish_kernel<<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, ws);
  }
  cut_hist_kernel<true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, use_k, ws);
  cut_gather_kernel<true, true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, use_k, 0ull, P, ws, da);
  sample_finish_kernel<true><<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, use_k, ws, da, out_tokens, out_logprobs, last_tok);
}

}  // namespace

void launch_sample(hipStream_t st, const float* logits, int M, int V, const RowMeta* rows, int pos_offset,
                   const int32_t* forced, float temperature, uint64_t seed, float* part, float* forced_z,
                   int32_t* out_tokens, float* out_logprobs, int top_k, float top_p, void* cut_buf, int32_t* last_tok) {
  const int n_tiles = (V + kSampleTile - 1) / kSampleTile;
  const int greedy = !(temperature > 0.f);
  const float inv_t = greedy ? 1.0f : 1.0f / temperature;
  const uint32_t seed_lo = (uint32_t)(seed & 0xffffffffu), seed_hi = (uint32_t)(seed >> 32);
  if (!greedy && sample_is_truncated(V, top_k, top_p)) {  // greedy ignores the cuts: the argmax is always kept
    launch_sample_cut(st, logits, M, V, inv_t, top_k, top_p, DrawArgs{rows, pos_offset, seed_lo, seed_hi, forced, forced_z, part},
                      (CutRow*)cut_buf, out_tokens, out_logprobs, last_tok);
    return;
  }
  if (V <= kSampleRowMax) {
    sample_row_kernel<<<M, std::min(1024, (V / 4 + 63) / 64 * 64), 0, st>>>(logits, V, rows, pos_offset, inv_t, greedy, seed_lo, seed_hi, forced,
                                                                            out_tokens, out_logprobs, last_tok);
    return;
  }
  sample_stage1_kernel<<<dim3(n_tiles, M), 256, 0, st>>>(logits, V, rows, pos_offset, inv_t, greedy, seed_lo, seed_hi, forced,
                                                         forced_z, part, n_tiles);
  sample_stage2_kernel<<<M, n_tiles <= 64 ? 64 : 1024, 0, st>>>(part, n_tiles, V, forced, forced_z, inv_t, out_tokens, out_logprobs, rows, last_tok);
}

void launch_sample_merge(hipStream_t st, const float* part, int n_tiles, int M, int V, const int32_t* forced,
                         const float* forced_z, float temperature, int32_t* out_tokens, float* out_logprobs,
                         const RowMeta* rows, int32_t* last_tok) {
  const float inv_t = temperature > 0.f ? 1.0f / temperature : 1.0f;
  sample_stage2_kernel<<<M, n_tiles <= 64 ? 64 : 1024, 0, st>>>(part, n_tiles, V, forced, forced_z, inv_t, out_tokens, out_logprobs, rows, last_tok);
}

}  // namespace rl

// ------------------------------------------------------------------------------------------------
// The plain sampler for callers that cannot allocate (code under graph capture, serving loops, harnesses that forbid
// it): the same kernels as above, with the row metadata, the forced tokens' logits and the per-tile partials in
// a file-scope device array instead of a model's workspace.  Each GPU has its own copy of the array at its own
// address; that address is looked up once per device and used from then on (the array's name is not a device
// address in host code).  Every call on a GPU uses that GPU's array, so calls that overlap on one GPU race.
// ------------------------------------------------------------------------------------------------
namespace rl {

namespace {

constexpr int kStaticRows = 256;          // rows per call
constexpr int kStaticTileRows = 20480;    // rows x ceil(vocab / kSampleTile) per call (151 936 entries x 256 rows: 19 200)
constexpr size_t kStaticRowsOff = 0;                                           // RowMeta [kStaticRows]
constexpr size_t kStaticForcedOff = kStaticRowsOff + kStaticRows * sizeof(RowMeta);  // float [kStaticRows]
constexpr size_t kStaticPartOff = kStaticForcedOff + kStaticRows * sizeof(float);    // float [kStaticTileRows][8]
constexpr size_t kStaticBytes = kStaticPartOff + (size_t)kStaticTileRows * kSamplePartFloats * sizeof(float);
static_assert(kStaticPartOff % 16 == 0, "the partials are written as float4");

static __device__ __align__(256) unsigned char scratch[kStaticBytes];  // 660 480 bytes per GPU, held until the process ends

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
unsigned char* g_scratch_ptr[kMaxDevices] = {};

// Address of the current device's copy of `scratch` (looked up on first use on that device).
hipError_t scratch_address(unsigned char** out) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (g_scratch_ptr[dev] == nullptr) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    g_scratch_ptr[dev] = (unsigned char*)p;
  }
  *out = g_scratch_ptr[dev];
  return hipSuccess;
}

__global__ __launch_bounds__(256) void static_rows_kernel(const int32_t* __restrict__ seq_ids, const int32_t* __restrict__ positions,
                                                          RowMeta* __restrict__ rows, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n) rows[i] = RowMeta{seq_ids[i], positions[i], 0, 0};
}

}  // namespace

}  // namespace rl

extern "C" rl_status rl_sample_logits_static(void* stream, int32_t n, int32_t vocab, const float* logits,
                                             const int32_t* seq_ids, const int32_t* positions, const int32_t* forced,
                                             const rl_sampling* sp, int32_t* out_tokens, float* out_logprobs) {
  using namespace rl;
  if (!logits || !seq_ids || !positions || !sp || !out_tokens || !out_logprobs)
    return (rl_status)set_error(RL_ERR_INVALID_ARG, "rl_sample_logits_static: NULL argument");
  if (vocab < 4 || vocab % 4 || vocab >= (1 << 22))
    return (rl_status)set_error(RL_ERR_INVALID_ARG, "rl_sample_logits_static: vocab %d must be a multiple of 4 in [4, 2^22)", vocab);
  const int n_tiles = (vocab + kSampleTile - 1) / kSampleTile;
  if (n < 1 || n > kStaticRows || (int64_t)n * n_tiles > kStaticTileRows)
    return (rl_status)set_error(RL_ERR_INVALID_ARG,
                                "rl_sample_logits_static: %d rows x %d vocabulary tiles exceed the static scratch "
                                "(at most %d rows and %d row-tiles of %d entries per call)",
                                n, n_tiles, kStaticRows, kStaticTileRows, kSampleTile);
  const int top_k = sp->top_k > (uint32_t)vocab ? 0 : (int)sp->top_k;
  if (sp->temperature > 0.f && sample_is_truncated(vocab, top_k, sp->top_p))
    return (rl_status)set_error(RL_ERR_UNSUPPORTED,
                                "rl_sample_logits_static: top-k / top-p cuts need per-row histograms that the static "
                                "scratch does not hold; use rl_sample_logits");
  unsigned char* base = nullptr;
  hipError_t e = scratch_address(&base);
  if (e != hipSuccess) return (rl_status)set_error(RL_ERR_DEVICE, "rl_sample_logits_static: scratch address: %s", hipGetErrorString(e));
  hipStream_t st = (hipStream_t)stream;
  RowMeta* rows = (RowMeta*)(base + kStaticRowsOff);
  float* forced_z = (float*)(base + kStaticForcedOff);
  float* part = (float*)(base + kStaticPartOff);
  // Nothing has to start at zero: the kernels write every entry they read (all n x n_tiles partials; the forced
  // token's logit whenever the forced id is inside the vocabulary, which is when the second stage reads it).
  static_rows_kernel<<<(n + 255) / 256, 256, 0, st>>>(seq_ids, positions, rows, n);
  launch_sample(st, logits, n, vocab, rows, 0, forced, sp->temperature, sp->seed, part, forced_z, out_tokens, out_logprobs);
  e = hipGetLastError();
  if (e != hipSuccess) return (rl_status)set_error(RL_ERR_DEVICE, "rl_sample_logits_static: %s", hipGetErrorString(e));
  return RL_OK;
}
