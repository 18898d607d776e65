// Stand-alone Gumbel-max sampling kernels (logits in memory) and the merge stage shared with the fused path.
// The arithmetic contract lives in sampler_device.h.  The log-probability log softmax(z/T)[token] is accumulated
// in fp32 (tolerance, not bit-exact).
#include <algorithm>
#include <mutex>

#include "../../include/rl.h"
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
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    best = better(best, shfl_xor_best(best, o));
    lse_merge(m, s, __shfl_xor(m, o, kWave), __shfl_xor(s, o, kWave));
  }
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
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    best = better(best, shfl_xor_best(best, o));
    lse_merge(m, s, __shfl_xor(m, o, kWave), __shfl_xor(s, o, kWave));
  }
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
//   1. cut_range: largest and smallest (finite) logit of the row.
//   2. cut_hist: count or integer mass per bin, the bins being kCutBins equal steps of the logit below the largest one --
//      over the 22 / inv_t in which weights are not zero for a mass, over the whole range for a count.  The bin is a
//      monotone function of the logit, so the bins are runs of the order, and integer masses make every sum exact.
//   3. cut_gather: every block redoes the scan of the histogram, which names the bin that holds the cut and what is still
//      to be covered inside it.  Tokens of earlier bins are certainly kept and take part in the draw at once; those of
//      the cut's bin (a few hundred at most over a row of logits) are collected in a list.
// sample_finish then finds the cut inside the list -- bins of the key between the list's smallest and largest, then a
// direct comparison of the tokens of one bin --, lets the list's kept tokens take part, and emits token and
// log-probability.  With both cuts, the count is selected first (passes 2, 3 and cut_finish) and the mass among what it
// keeps.  Rows whose list overflows (thousands of tokens within a thousandth of the range) or whose largest score is not
// a number of ordinary size are selected by one block digit by digit instead (radix_cut).
// A radix selection over the row's key digits took five passes, each with its own scan: 217 us for 128 rows of 151936
// entries at 0.6 / 0.95, of which 151 us were these passes and 37 us a draw over every entry; now 76 us.
// ------------------------------------------------------------------------------------------------
constexpr int kCutBins = 1024;
constexpr int kCutList = 4096;
constexpr int kCutThreads = 512;
constexpr int kCutSlices = 32;  // at most, per row
constexpr int kRadixBins = 2048;

struct CutSel {            // after the scan of a histogram
  int32_t bin;             // the bin that holds the cut
  int32_t pad;
  unsigned long long rem;  // count or mass still to be covered inside it
};
struct CutRow {  // per row
  unsigned long long hist[2][kCutBins];  // selection 0: count (top-k), 1: mass (top-p)
  CutSel sel[2];
  uint32_t n_list[2];                    // tokens that asked for a place in the list
  OrderCut cut_k;
  uint32_t kmax[kCutSlices], kmin[kCutSlices];  // per slice: largest key; smallest key of a finite logit (or 0xffffffff)
  uint2 list[2][kCutList];               // (key, index)
};
static_assert(sizeof(CutRow) % 16 == 0, "rows lie one behind the other, histograms are read in pairs");

// Calls fn(i, z[i]) for the tokens of float4 groups [g_begin, g_end) of the row (V % 4 == 0, rows 16-byte aligned),
// four 16-byte loads in flight per thread.
template <typename F>
__device__ __forceinline__ void for_each_group(const float* __restrict__ z, int g_begin, int g_end, int tid, int nthr, F fn) {
  for (int g0 = g_begin + tid; g0 < g_end; g0 += 4 * nthr) {
    float4 v[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int g = g0 + e * nthr;
      v[e] = g < g_end ? ((const float4*)z)[g] : make_float4(0.f, 0.f, 0.f, 0.f);
    }
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int g = g0 + e * nthr;
      if (g < g_end) fn(4 * g, v[e]);
    }
  }
}
template <typename F>
__device__ __forceinline__ void for_each_token(const float* __restrict__ z, int g_begin, int g_end, int tid, int nthr, F fn) {
  for_each_group(z, g_begin, g_end, tid, nthr, [&](int i, float4 v) { fn(i, v.x); fn(i + 1, v.y); fn(i + 2, v.z); fn(i + 3, v.w); });
}

__device__ __forceinline__ bool finite_bits(float x) { return (__float_as_uint(x) & 0x7f800000u) != 0x7f800000u; }

struct Slice { int g_begin, g_end; };
__device__ __forceinline__ Slice row_slice(int V) {
  const int n4 = V >> 2, per = (n4 + gridDim.x - 1) / gridDim.x;
  const int g = min(n4, (int)blockIdx.x * per);
  return Slice{g, min(n4, g + per)};
}

// The row's largest logit, and the bins of a selection.
struct CutBinning {
  float z_max, s_max;  // largest logit; the same times 1/T
  float scale;         // bins per unit of the logit
  bool ok;             // the largest score is finite ...
  __device__ __forceinline__ int bin(float z) const { return (int)fminf((z_max - z) * scale, (float)(kCutBins - 1)); }
};
__device__ __forceinline__ CutBinning cut_binning(const CutRow& row, int n_slices, float inv_t, bool mass) {
  uint32_t kmax = 0, kmin = 0xffffffffu;
  for (int i = 0; i < n_slices; ++i) {  // the same addresses for every lane
    kmax = max(kmax, row.kmax[i]);
    kmin = min(kmin, row.kmin[i]);
  }
  CutBinning b;
  b.z_max = order_value(kmax);
  b.s_max = __fmul_rn(b.z_max, inv_t);
  // ... and known well enough that the largest logit's own weight is about 2^32 (scores beyond 10^7 round by more)
  const float x0 = __fmaf_rn(b.z_max, inv_t, -b.s_max);
  b.ok = finite_bits(b.z_max) && finite_bits(b.s_max) && finite_bits(inv_t) && x0 > -1.f && x0 < 0.3f;
  float range = b.z_max - order_value(min(kmin, kmax));
  if (mass) range = fminf(range, 22.5f / inv_t);
  b.scale = range > 0.f ? (float)(kCutBins - 1) / range : 0.f;
  if (!finite_bits(b.scale)) b.scale = 0.f;  // a range below 2^-118: one bin
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

// grid (slices, rows): the slice's largest and smallest finite key; clears the row's histograms and counters.
__global__ __launch_bounds__(kCutThreads) void cut_range_kernel(const float* __restrict__ logits, int V, CutRow* __restrict__ ws) {
  __shared__ uint32_t sh[2][kCutThreads / 64];
  const int r = blockIdx.y, tid = threadIdx.x;
  CutRow& row = ws[r];
  for (int i = blockIdx.x * kCutThreads + tid; i < 2 * kCutBins; i += gridDim.x * kCutThreads) (&row.hist[0][0])[i] = 0ull;
  if (blockIdx.x == 0 && tid < 2) row.n_list[tid] = 0u;
  const Slice sl = row_slice(V);
  uint32_t kmax = 0, kmin = 0xffffffffu;
  for_each_token(logits + (size_t)r * V, sl.g_begin, sl.g_end, tid, kCutThreads, [&](int, float zi) {
    const uint32_t k = order_key(zi);
    kmax = max(kmax, k);
    kmin = min(kmin, finite_bits(zi) ? k : 0xffffffffu);
  });
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    kmax = max(kmax, (uint32_t)__shfl_xor((int)kmax, o, kWave));
    kmin = min(kmin, (uint32_t)__shfl_xor((int)kmin, o, kWave));
  }
  if ((tid & 63) == 0) { sh[0][tid >> 6] = kmax; sh[1][tid >> 6] = kmin; }
  __syncthreads();
  if (tid == 0) {
    for (int w = 1; w < kCutThreads / 64; ++w) { kmax = max(kmax, sh[0][w]); kmin = min(kmin, sh[1][w]); }
    row.kmax[blockIdx.x] = kmax;
    row.kmin[blockIdx.x] = kmin;
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
  if (!cb.ok) return;  // block-uniform: sample_finish takes the row
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  for (int b = tid; b < kCutBins; b += kCutThreads) lh[b] = 0ull;
  __syncthreads();
  const Slice sl = row_slice(V);
  for_each_token(logits + (size_t)r * V, sl.g_begin, sl.g_end, tid, kCutThreads, [&](int i, float zi) {
    unsigned long long w = 1ull;
    if (kMass) {
      const float x = __fmaf_rn(zi, inv_t, -cb.s_max);
      if (!(x > -22.0f)) return;  // weight zero
      w = fexp_weight(x);
    }
    if (use_k && !kept_by(allowed, order_key(zi), i)) return;
    atomicAdd(&lh[cb.bin(zi)], w);
  });
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
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    d.best = better(d.best, shfl_xor_best(d.best, o));
    d.sum = Draw::plus(d.sum, __shfl_xor(d.sum, o, kWave));
  }
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
// earlier bins.  The draw's partials are written even where the row goes to radix_cut (and are not read there).
template <bool kMass, bool kDraw>
__global__ __launch_bounds__(kCutThreads) void cut_gather_kernel(const float* __restrict__ logits, int V, float inv_t, int use_k,
                                                                 unsigned long long target, unsigned long long p_fixed,
                                                                 CutRow* __restrict__ ws, DrawArgs da) {
  constexpr int kOwn = 1024;  // a block's own list, so that the row's counter sees one addition per block
  __shared__ CutSel sh_sel;
  __shared__ Draw sh_draw[kCutThreads / 64];
  constexpr int kKept = kDraw ? 2048 : 1;  // certainly kept tokens, drawn among after the scan with all lanes busy
  __shared__ uint2 sh_list[kOwn], sh_kept[kKept];
  __shared__ uint32_t sh_n, sh_at, sh_nk;
  const int r = blockIdx.y, tid = threadIdx.x;
  CutRow& row = ws[r];
  const CutBinning cb = cut_binning(row, gridDim.x, inv_t, kMass);
  if (!cb.ok) return;  // block-uniform: sample_finish takes the row
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  if (tid < 64) {
    const unsigned long long* h = row.hist[kMass];
    CutSel sel{0, 0, 0ull};
    sel.bin = scan_select_n<false, kCutBins / 64>(h, [&](unsigned long long S) { return kMass ? mass_target(S, p_fixed) : target; }, tid, &sel.rem);
    if (tid == 0) {
      sh_sel = sel;
      sh_n = sh_nk = 0u;
      if (blockIdx.x == 0) row.sel[kMass] = sel;
    }
  }
  __syncthreads();
  const int cut_bin = sh_sel.bin;
  const float* z = logits + (size_t)r * V;
  const Slice sl = row_slice(V);
  uint32_t pos = 0, seq = 0;
  int f = -1;
  if (kDraw) {
    const RowMeta rm = da.rows[r];
    pos = (uint32_t)(rm.pos + da.pos_offset);
    seq = (uint32_t)rm.seq;
    if (da.forced) f = da.forced[r];
  }
  Draw d = empty_draw();
  auto draw_token = [&](int i, float zi) {
    d.add(i, zi, cb.z_max, inv_t, token_bits((uint32_t)i, pos, seq, da.seed_lo, da.seed_hi));
  };
  auto put = [&](uint32_t at, uint2 e) { if (at < (uint32_t)kCutList) row.list[kMass][at] = e; };
  for_each_group(z, sl.g_begin, sl.g_end, tid, kCutThreads, [&](int i0, float4 v) {
    const float zs[4] = {v.x, v.y, v.z, v.w};
    // most groups lie behind the cut's bin as a whole
    const float top = fmaxf(fmaxf(v.x, v.y), fmaxf(v.z, v.w));
    const bool any = cb.bin(top) <= cut_bin;  // a NaN is the largest key (row not ok) or the smallest: fmaxf skips it
    if (kDraw && !any && f >= i0 && f < i0 + 4) da.forced_z[r] = -INFINITY;  // cut off: probability zero
    if (!any) return;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int b = cb.bin(zs[e]);
      const uint32_t k = order_key(zs[e]);
      if (b > cut_bin || (use_k && !kept_by(allowed, k, i0 + e))) {
        if (kDraw && f == i0 + e) da.forced_z[r] = -INFINITY;
        continue;
      }
      if (b == cut_bin) {
        if (kDraw && f == i0 + e) da.forced_z[r] = -INFINITY;  // unless sample_finish keeps it
        if (kMass && !(__fmaf_rn(zs[e], inv_t, -cb.s_max) > -22.0f)) continue;  // weight zero: never the cut, always behind it
        const uint32_t at = atomicAdd(&sh_n, 1u);
        if (at < (uint32_t)kOwn) sh_list[at] = make_uint2(k, (uint32_t)(i0 + e));
        else put(atomicAdd(&row.n_list[kMass], 1u), make_uint2(k, (uint32_t)(i0 + e)));
        continue;
      }
      if (kDraw) {
        const uint32_t at = atomicAdd(&sh_nk, 1u);
        if (at < (uint32_t)kKept) sh_kept[at] = make_uint2(__float_as_uint(zs[e]), (uint32_t)(i0 + e));
        else draw_token(i0 + e, zs[e]);
        if (f == i0 + e) da.forced_z[r] = zs[e];
      }
    }
  });
  __syncthreads();
  const uint32_t n_own = min(sh_n, (uint32_t)kOwn);
  if (tid == 0 && n_own > 0) sh_at = atomicAdd(&row.n_list[kMass], n_own);
  __syncthreads();
  for (uint32_t t = tid; t < n_own; t += kCutThreads) put(sh_at + t, sh_list[t]);
  if (!kDraw) return;
  for (uint32_t t = tid; t < min(sh_nk, (uint32_t)kKept); t += kCutThreads) draw_token((int)sh_kept[t].y, __uint_as_float(sh_kept[t].x));
  d = block_draw<kCutThreads>(d, sh_draw);
  if (tid == 0) {
    float* p = da.part + ((size_t)r * gridDim.x + blockIdx.x) * kSamplePartFloats;
    *(float4*)p = make_float4(d.best.y, __int_as_float(d.best.idx), d.best.z, 0.f);
    *(unsigned long long*)(p + 4) = d.sum;
  }
}

// Four (bin, count-or-mass) entries in registers.  The top digit of the order key takes only a handful of values over
// a row of logits, so in the first stage nearly every token would hit the same few LDS words; a thread collects them
// here and adds each entry to the histogram once.
struct BinCache {
  int bin[4];
  unsigned long long val[4];
  int next;
  __device__ __forceinline__ void init() {
#pragma unroll
    for (int e = 0; e < 4; ++e) { bin[e] = -1; val[e] = 0; }
    next = 0;
  }
  __device__ __forceinline__ void add(int b, unsigned long long w, unsigned long long* h) {
    bool hit = false;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (bin[e] == b) { val[e] += w; hit = true; }
    if (hit) return;
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (next == e) {
        if (bin[e] >= 0) atomicAdd(&h[bin[e]], val[e]);
        bin[e] = b;
        val[e] = w;
      }
    next = (next + 1) & 3;
  }
  __device__ __forceinline__ void flush(unsigned long long* h) {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (bin[e] >= 0) atomicAdd(&h[bin[e]], val[e]);
  }
};

constexpr int kFinishThreads = 1024;
struct FinishLds {
  __align__(16) unsigned long long hist[kRadixBins];
  uint2 list[kCutList];
  Draw draw[kFinishThreads / 64];
  unsigned long long rem;
  uint32_t lo, hi, n;
  OrderCut cut;
};

// The cut of a whole row by one block, digit by digit of the order key from the top (11, 11, 10 bits) and then of the
// index (11, 11 bits, ascending) among the tokens that share the cut's key: count or mass per digit, scanned until the
// target is reached.  Any row, whatever its values.  Every thread returns the cut.
template <bool kMass>
__device__ OrderCut radix_cut(const float* __restrict__ z, int V, float inv_t, float s_max, unsigned long long target,
                              unsigned long long p_fixed, OrderCut allowed, FinishLds& sh) {
  const int tid = threadIdx.x, lane = tid & 63;
  uint32_t prefix = 0, iprefix = 0;
  unsigned long long rem = target;
  for (int stage = 0; stage < 5; ++stage) {
    const int shift = stage == 0 ? 21 : stage == 1 ? 10 : stage == 2 ? 0 : stage == 3 ? 11 : 0;
    const int width = stage == 2 ? 10 : 11;
    const uint32_t mask = (1u << width) - 1;
    __syncthreads();
    for (int b = tid; b < kRadixBins; b += kFinishThreads) sh.hist[b] = 0ull;
    __syncthreads();
    if (stage == 0) {
      BinCache bc;
      bc.init();
      for_each_token(z, 0, V >> 2, tid, kFinishThreads, [&](int i, float zi) {
        const uint32_t k = order_key(zi);
        if (!kept_by(allowed, k, i)) return;
        bc.add((int)(k >> shift), kMass ? fexp_weight(__fmaf_rn(zi, inv_t, -s_max)) : 1ull, sh.hist);
      });
      bc.flush(sh.hist);
    } else {
      for_each_token(z, 0, V >> 2, tid, kFinishThreads, [&](int i, float zi) {
        const uint32_t k = order_key(zi);
        if (!kept_by(allowed, k, i)) return;
        if (stage < 3) {
          if ((k >> (shift + width)) != (prefix >> (shift + width))) return;
          atomicAdd(&sh.hist[(k >> shift) & mask], kMass ? fexp_weight(__fmaf_rn(zi, inv_t, -s_max)) : 1ull);
        } else {
          if (k != prefix || (stage == 4 && ((uint32_t)i >> 11) != (iprefix >> 11))) return;
          atomicAdd(&sh.hist[((uint32_t)i >> shift) & mask], 1ull);
        }
      });
    }
    __syncthreads();
    const auto covered = [&](unsigned long long S) { return kMass && stage == 0 ? mass_target(S, p_fixed) : rem; };
    unsigned long long rem_out;  // the same in every wave
    if (stage < 3) {
      const int b = stage == 2 ? scan_select_n<true, 16>(sh.hist, covered, lane, &rem_out) : scan_select_n<true, 32>(sh.hist, covered, lane, &rem_out);
      prefix |= (uint32_t)b << shift;
      if (stage == 2) {  // key complete: tokens with this key, in ascending index order -- how many are needed
        if (kMass) {
          const unsigned long long w = fexp_weight(__fmaf_rn(order_value(prefix), inv_t, -s_max));
          rem_out = w > 0 ? (rem_out + w - 1) / w : 1ull;
        }
        if (rem_out < 1) rem_out = 1;
      }
    } else {
      iprefix |= (uint32_t)scan_select_n<false, 32>(sh.hist, covered, lane, &rem_out) << shift;
    }
    rem = rem_out;
  }
  __syncthreads();
  return OrderCut{prefix, (int32_t)iprefix};
}

// The cut inside the n listed tokens of its bin, of whose count or mass `rem` is to be covered: equal steps of the key
// between the smallest and the largest, then the tokens of one step against each other.  False where a step holds more
// than kCutFew tokens.  Leaves the list in sh.list.
constexpr int kCutFew = 512;
static_assert(kCutFew <= kFinishThreads && kCutFew <= kCutBins, "one thread each, in half of the histogram's place");
template <bool kMass>
__device__ bool list_cut(const uint2* __restrict__ list, int n, unsigned long long rem, float inv_t, float s_max, FinishLds& sh,
                         OrderCut* cut) {
  const int tid = threadIdx.x, lane = tid & 63;
  if (tid == 0) { sh.lo = 0xffffffffu; sh.hi = 0u; sh.n = 0u; }
  for (int b = tid; b < kCutBins; b += kFinishThreads) sh.hist[b] = 0ull;
  __syncthreads();
  uint32_t lo = 0xffffffffu, hi = 0u;
  for (int t = tid; t < n; t += kFinishThreads) {
    const uint2 e = list[t];
    sh.list[t] = e;
    lo = min(lo, e.x);
    hi = max(hi, e.x);
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    lo = min(lo, (uint32_t)__shfl_xor((int)lo, o, kWave));
    hi = max(hi, (uint32_t)__shfl_xor((int)hi, o, kWave));
  }
  if (lane == 0) { atomicMin(&sh.lo, lo); atomicMax(&sh.hi, hi); }
  __syncthreads();
  hi = sh.hi;
  const uint32_t span = hi - sh.lo;
  const int shift = max(0, 32 - (int)__clz((int)span) - 10);  // span >> shift < kCutBins
  auto weight = [&](uint32_t k) { return kMass ? fexp_weight(__fmaf_rn(order_value(k), inv_t, -s_max)) : 1ull; };
  for (int t = tid; t < n; t += kFinishThreads) atomicAdd(&sh.hist[(hi - sh.list[t].x) >> shift], weight(sh.list[t].x));
  __syncthreads();
  unsigned long long left;
  const uint32_t bin = (uint32_t)scan_select_n<false, kCutBins / 64>(sh.hist, [&](unsigned long long) { return rem; }, lane, &left);  // the same in every wave
  // the tokens of that step and their weights, in the place of the histogram: the cut is the one whose own weight
  // reaches what is left
  uint2* const few = (uint2*)(sh.hist + kCutBins);
  unsigned long long* const few_w = sh.hist;
  __syncthreads();
  for (int t = tid; t < n; t += kFinishThreads)
    if (((hi - sh.list[t].x) >> shift) == bin) {
      const uint32_t at = atomicAdd(&sh.n, 1u);
      if (at < (uint32_t)kCutFew) { few[at] = sh.list[t]; few_w[at] = weight(sh.list[t].x); }
    }
  __syncthreads();
  const int n_few = (int)sh.n;
  if (n_few > kCutFew) return false;  // block-uniform
  if (tid < n_few) {
    const uint2 e = few[tid];
    unsigned long long before = 0;
    for (int u = 0; u < n_few; ++u) {
      const uint2 o = few[u];
      if (o.x > e.x || (o.x == e.x && o.y < e.y)) before += few_w[u];
    }
    if (before < left && left <= before + few_w[tid]) sh.cut = OrderCut{e.x, (int32_t)e.y};  // exactly one token
  }
  __syncthreads();
  *cut = sh.cut;
  return true;
}

// The row's cut of selection kMass, in every thread: from its list where that holds it, otherwise from the whole row.
// Returns whether it came from the list, which is then in sh.list.
template <bool kMass>
__device__ bool row_cut(const float* __restrict__ z, int V, float inv_t, const CutBinning& cb, const CutRow& row,
                        unsigned long long target, unsigned long long p_fixed, OrderCut allowed, FinishLds& sh, OrderCut* cut) {
  const uint32_t n = row.n_list[kMass];
  if (cb.ok && n <= (uint32_t)kCutList && list_cut<kMass>(row.list[kMass], (int)n, row.sel[kMass].rem, inv_t, cb.s_max, sh, cut)) return true;
  *cut = radix_cut<kMass>(z, V, inv_t, cb.s_max, target, p_fixed, allowed, sh);
  return false;
}

// grid (rows): the top-k cut of a row that a top-p cut will follow.
__global__ __launch_bounds__(kFinishThreads) void cut_finish_kernel(const float* __restrict__ logits, int V, float inv_t, int n_slices,
                                                                    unsigned long long target, CutRow* __restrict__ ws) {
  __shared__ FinishLds sh;
  CutRow& row = ws[blockIdx.x];
  const CutBinning cb = cut_binning(row, n_slices, inv_t, false);
  OrderCut cut;
  row_cut<false>(logits + (size_t)blockIdx.x * V, V, inv_t, cb, row, target, 0ull, OrderCut{0u, 0x7fffffff}, sh, &cut);
  if (threadIdx.x == 0) row.cut_k = cut;
}

// grid (rows): the final cut, the draw among the tokens of its bin, and the result.
template <bool kMass>
__global__ __launch_bounds__(kFinishThreads) void sample_finish_kernel(const float* __restrict__ logits, int V, float inv_t,
                                                                       int n_slices, int use_k, unsigned long long target,
                                                                       unsigned long long p_fixed, const CutRow* __restrict__ ws,
                                                                       DrawArgs da, int32_t* __restrict__ out_tok,
                                                                       float* __restrict__ out_lp, int32_t* __restrict__ last_tok) {
  __shared__ FinishLds sh;
  const int r = blockIdx.x, tid = threadIdx.x;
  const CutRow& row = ws[r];
  const float* z = logits + (size_t)r * V;
  const CutBinning cb = cut_binning(row, n_slices, inv_t, kMass);
  const OrderCut allowed = use_k ? row.cut_k : OrderCut{0u, 0x7fffffff};
  const RowMeta rm = da.rows[r];
  const uint32_t pos = (uint32_t)(rm.pos + da.pos_offset), seq = (uint32_t)rm.seq;
  const int f = da.forced ? da.forced[r] : -1;
  __shared__ float sh_fz;
  Draw d = empty_draw();
  if (tid == 0 && f >= 0 && f < V) sh_fz = da.forced_z[r];
  OrderCut cut;
  if (!row_cut<kMass>(z, V, inv_t, cb, row, target, p_fixed, allowed, sh, &cut)) {
    for_each_group(z, 0, V >> 2, tid, kFinishThreads, [&](int i0, float4 v) {
      const float zs[4] = {v.x, v.y, v.z, v.w};
      uint32_t rnd[4];
      philox4x32_10((uint32_t)i0 >> 2, pos, seq, 0u, da.seed_lo, da.seed_hi, rnd);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const bool kept = kept_by(cut, order_key(zs[e]), i0 + e);
        if (i0 + e == f) sh_fz = kept ? zs[e] : -INFINITY;
        if (kept) d.add(i0 + e, zs[e], cb.z_max, inv_t, rnd[e]);
      }
    });
  } else {
    for (int t = tid; t < (int)row.n_list[kMass]; t += kFinishThreads) {
      const uint2 e = sh.list[t];
      if (!kept_by(cut, e.x, (int)e.y)) continue;
      const float zi = order_value(e.x);
      d.add((int)e.y, zi, cb.z_max, inv_t, token_bits(e.y, pos, seq, da.seed_lo, da.seed_hi));
      if ((int)e.y == f) sh_fz = zi;
    }
    for (int t = tid; t < n_slices; t += kFinishThreads) {
      const float* p = da.part + ((size_t)r * n_slices + t) * kSamplePartFloats;
      Draw o;
      o.best = Best{p[0], __float_as_int(p[1]), p[2]};
      o.sum = *(const unsigned long long*)(p + 4);
      d.merge(o);
    }
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
  // About two blocks per compute unit: every block clears, scans or flushes a histogram of its own (at 128 rows 4 slices
  // of 512 threads 76 us, 8 slices 81, 4 of 1024 threads 77, 16 of 256 threads 90).
  int slices = 512 / M;
  slices = std::max(1, std::min(std::min(slices, kCutSlices), (V + kSampleTile - 1) / kSampleTile));
  const dim3 grid(slices, M);
  cut_range_kernel<<<grid, kCutThreads, 0, st>>>(logits, V, ws);
  if (use_k) {
    cut_hist_kernel<false><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, ws);
    if (!use_p) {
      cut_gather_kernel<false, true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, K, 0ull, ws, da);
      sample_finish_kernel<false><<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, 0, K, 0ull, ws, da, out_tokens, out_logprobs, last_tok);
      return;
    }
    cut_gather_kernel<false, false><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, 0, K, 0ull, ws, da);
    cut_finish_kernel<<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, K, ws);
  }
  cut_hist_kernel<true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, use_k, ws);
  cut_gather_kernel<true, true><<<grid, kCutThreads, 0, st>>>(logits, V, inv_t, use_k, 0ull, P, ws, da);
  sample_finish_kernel<true><<<M, kFinishThreads, 0, st>>>(logits, V, inv_t, slices, use_k, 1ull, P, ws, da, out_tokens, out_logprobs, last_tok);
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
// it): the same two kernels as above, with the row metadata, the forced tokens' logits and the per-tile partials in
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
