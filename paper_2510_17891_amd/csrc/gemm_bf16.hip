// Weight-streaming bf16 GEMM for decode-sized batches:  Y[M x N] = X[M x K] * W[N x K]^T.
//
// At M <= 256 the projection is bound by reading W once from HBM (M flop per weight byte), so the kernel is
// organised around that stream: both operands are stored fragment-major (see frag_offset), which makes every
// global load a fully coalesced 1 KiB wave access that lands directly in MFMA 32x32x16 operand registers (the packed
// weights hold the f16 image of the model's bf16 weights; the activations arrive as f16) -- no LDS staging, no shuffles.  A wave owns a 64 x (32*MB) output tile over a slice of K; the four waves of a
// block take four K slices and add their accumulators through LDS in a fixed order; further K splits across
// blocks (to put >= 256 blocks on the chip for the small matrices) leave fp32 partials that the consumer sums.
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"
#include "sampler_device.h"

namespace rl {

namespace {

typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));

__device__ __forceinline__ f32x16_t mfma_f16(u32x4_t a, u32x4_t b, f32x16_t c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0, 0, 0);
}

template <int MB, int RB = 2>
struct Frags {
  u32x4_t a[RB][4];  // RB 32-row blocks of the weight matrix
  u32x4_t b[MB][4];
};

// wr[nb]: row block nb of the tile; NT: weights pass through once (non-temporal), otherwise the block's other waves
// read the same tile and it may live in L1/L2.
// kb: the k block (activations are stored in that order); kw: where the weights keep it (weight_kb_slot).
template <int MB, int RB, bool NT = true>
__device__ __forceinline__ void load_frags(Frags<MB, RB>& f, const u32x4_t* const (&wr)[RB],
                                           const u32x4_t* const* __restrict__ xb, int kb, int kw, int lane) {
  // block (rb, slot) = 256 uint4; sub-load t is [t*64 + lane]
  const int o = kb * 256 + lane, ow = kw * 256 + lane;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) f.a[nb][t] = NT ? __builtin_nontemporal_load(wr[nb] + ow + t * 64) : wr[nb][ow + t * 64];
  }
#pragma unroll
  for (int mb = 0; mb < MB; ++mb)
#pragma unroll
    for (int t = 0; t < 4; ++t) f.b[mb][t] = xb[mb][o + t * 64];
}

template <int MB, int RB>
__device__ __forceinline__ void mma_frags(const Frags<MB, RB>& f, f32x16_t (&acc)[RB][MB]) {
#pragma unroll
  for (int t = 0; t < 4; ++t)
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) {
      const u32x4_t a = f.a[nb][t];
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) acc[nb][mb] = mfma_f16(a, f.b[mb][t], acc[nb][mb]);
    }
}

// One finished 32-row block held in MFMA accumulator order -- lane (col, hb) has outputs 8q + 4hb + e (q, e = 0..3)
// of batch row m -- for the epilogues that work per row block.
template <int EPI>
__device__ __forceinline__ void store_rowblock(const float (&sum)[16], int m, int hb, int rb, int split, int M, int N,
                                               void* __restrict__ out) {
  if (EPI == kEpiPartial) {
    float* o = (float*)out + ((size_t)split * M + m) * N;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      *(float4*)(o + rb * 32 + 8 * q + 4 * hb) = make_float4(sum[4 * q], sum[4 * q + 1], sum[4 * q + 2], sum[4 * q + 3]);
  } else {
    // SwiGLU: a 32-row block of the interleaved gate/up matrix holds the gate rows (0..15) and the up rows (16..31)
    // of the 16 outputs 16 rb .. 16 rb + 15: a lane finds both factors of its outputs in its own registers.
    uint16_t* o = (uint16_t*)out;
#pragma unroll
    for (int q = 0; q < 2; ++q) {
      float a[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float gte = sum[4 * q + e], up = sum[4 * (q + 2) + e];
        a[e] = gte / (1.0f + __expf(-gte)) * up;
      }
      *(uint2*)(o + frag_offset(m, rb * 16 + 8 * q + 4 * hb, N >> 6)) = make_uint2(pack2h(a[0], a[1]), pack2h(a[2], a[3]));
    }
  }
}

// Write one finished 64 x 32 output block held in MFMA accumulator order: lane (col, hb) has, for both row blocks,
// outputs n = rb*32 + 8q + 4hb + e (q, e = 0..3) of batch row m.
template <int EPI>
__device__ __forceinline__ void store_block(const float (&sum)[2][16], int m, int hb, int rb0, int rb1, int split, int M,
                                          int N, void* __restrict__ out, const SampleEpilogue& se, int tile) {
  if (EPI == kEpiPartial || EPI == kEpiSwiGLU) {
    store_rowblock<EPI>(sum[0], m, hb, rb0, split, M, N, out);
    store_rowblock<EPI>(sum[1], m, hb, rb1, split, M, N, out);
  } else {
    // lane (col, hb) holds 32 logits of row m: vocabulary ids (rb*32 + 8q + 4hb + e), in aligned groups of four,
    // i.e. one Philox block per group.
    const RowMeta rm = se.rows[m];
    const uint32_t pos = (uint32_t)(rm.pos + se.pos_offset), seq = (uint32_t)rm.seq;
    const int f = se.forced ? se.forced[m] : -1;
    Best best{-INFINITY, -1, 0.f};
    // log-sum-exp of the lane's 32 entries: their maximum first, then one exponential per entry
    float lm = -INFINITY, ls = 0.f;
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) lm = fmaxf(lm, sum[nb][r] * se.inv_t);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int n0 = (nb ? rb1 : rb0) * 32 + 8 * q + 4 * hb;
        uint32_t rnd[4] = {0, 0, 0, 0};
        if (!se.greedy) philox4x32_10((uint32_t)n0 >> 2, pos, seq, 0u, se.seed_lo, se.seed_hi, rnd);
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float zi = sum[nb][4 * q + e];
          const float y = se.greedy ? zi : __fmaf_rn(zi, se.inv_t, gumbel(rnd[e]));
          best = better(best, Best{y, n0 + e, zi});
          if (lm != -INFINITY) ls += __expf(zi * se.inv_t - lm);
          if (n0 + e == f) se.forced_z[m] = zi;
        }
        if (se.logits_out)
          *(float4*)(se.logits_out + (size_t)m * N + n0) =
              make_float4(sum[nb][4 * q], sum[nb][4 * q + 1], sum[nb][4 * q + 2], sum[nb][4 * q + 3]);
      }
    best = best_of_lanes(best, 32);  // the other half of this row's 64 entries
    lse_merge_lanes(lm, ls, 32);
    if (hb == 0) {
      float* p = se.part + ((size_t)m * (N >> 6) + tile) * kSamplePartFloats;
      *(float4*)p = make_float4(best.y, __int_as_float(best.idx), best.z, 0.f);
      *(float4*)(p + 4) = make_float4(lm, ls, 0.f, 0.f);
    }
  }
}

// grid: x = N tile, y = K split, z = M tile of 32*MB rows.
//   EPI == kEpiPartial: tile = 64 output columns (row blocks 2x, 2x+1 of W); out fp32 [S][M][N].
//   EPI == kEpiSwiGLU : tile = 32 output columns (row blocks 2x, 2x+1 of the interleaved gate/up matrix, each 16 gate
//                       rows and the 16 up rows of the same outputs); out f16 fragment-major [M x N].
//   EPI == kEpiSample : tile = 64 vocabulary entries; the logits stay in registers: temperature, Gumbel noise, running
//                       arg-max and log-sum-exp are taken per (row, tile) and only those partials are written
//                       (plus the logits themselves when the caller asked for them).
// ST = k blocks a wave keeps in flight.  HBM latency is ~10x the MFMA time of a block, so the loop is a ring of
// ST register buffers: compute block i, immediately re-issue its buffer for block i + ST.  The scheduling
// barriers keep the compiler from sinking the loads below the next block's MFMAs.
// One tile of RB 32-row blocks (rb_first .. rb_first + RB - 1) over the K range of `split`, for batch tile m_tile:
// the body of the K-split kernels.  `tile` is the index of the 64-entry vocabulary tile (sampling epilogue, RB == 2).
template <int MB, int EPI, int ST, int RB>
__device__ __forceinline__ void kslice_tile(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                            void* __restrict__ out, int M, int N, int K, int kb_per_wave,
                                            const SampleEpilogue& se, int rb_first, int split, int m_tile, int tile,
                                            float (&red)[4][16][64]) {
  static_assert(EPI != kEpiSample || RB == 2, "the sampling epilogue works on 64-entry tiles");
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int KB = K >> 6;
  const int m_blk0 = m_tile * MB;
  const int n_blocks_m = (M + 31) >> 5;
  const u32x4_t* wr[RB];
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) wr[nb] = W + (size_t)(rb_first + nb) * KB * 256;
  const u32x4_t* xb[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    int b = m_blk0 + mb;
    if (b >= n_blocks_m) b = n_blocks_m - 1;  // clamp: surplus column blocks are computed but never stored
    xb[mb] = X + (size_t)b * KB * 256;
  }

  f32x16_t acc[RB][MB];
#pragma unroll
  for (int nb = 0; nb < RB; ++nb)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[nb][mb][r] = 0.f;

  const int kb0 = (split * 4 + wave) * kb_per_wave;
  const int kw0 = split * 4 * kb_per_wave + wave;  // slot of k block kb0; this wave's later blocks follow at stride 4
  const int n = kb_per_wave;
  Frags<MB, RB> f[ST];
#pragma unroll
  for (int s = 0; s < ST; ++s) load_frags<MB, RB>(f[s], wr, xb, kb0 + s, kw0 + 4 * s, lane);  // the launcher guarantees ST <= n
  const int full = n / ST, rem = n - full * ST;
  int b = 0;
  for (int r = 0; r + 1 < full; ++r) {  // steady state: every buffer is refilled
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      mma_frags<MB, RB>(f[s], acc);
      __builtin_amdgcn_sched_barrier(0);
      load_frags<MB, RB>(f[s], wr, xb, kb0 + b + s + ST, kw0 + 4 * (b + s + ST), lane);
      __builtin_amdgcn_sched_barrier(0);
    }
    b += ST;
  }
  if (full > 0) {  // last full round: refill only what the remainder round will use
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      mma_frags<MB, RB>(f[s], acc);
      __builtin_amdgcn_sched_barrier(0);
      if (s < rem) load_frags<MB, RB>(f[s], wr, xb, kb0 + b + s + ST, kw0 + 4 * (b + s + ST), lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < rem) mma_frags<MB, RB>(f[s], acc);

  // ---- add the four waves' accumulators (fixed order) and write: column block mb is finished by wave mb % 4 ----
  const int col = lane & 31, hb = lane >> 5;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    float sum[RB][16];
#pragma unroll
    for (int nb = 0; nb < RB; ++nb) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[nb][mb][r];
      __syncthreads();
      if (wave == (mb & 3)) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          sum[nb][r] = ((red[0][r][lane] + red[1][r][lane]) + red[2][r][lane]) + red[3][r][lane];
      }
    }
    if (wave != (mb & 3)) continue;
    const int m = (m_blk0 + mb) * 32 + col;
    if (m >= M) continue;
    if constexpr (EPI == kEpiSample) {
      store_block<EPI>(sum, m, hb, rb_first, rb_first + 1, split, M, N, out, se, tile);
    } else {
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) store_rowblock<EPI>(sum[nb], m, hb, rb_first + nb, split, M, N, out);
    }
  }
}

template <int MB, int EPI, int ST>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                        void* __restrict__ out, int M, int N, int K, int kb_per_wave,
                                                        SampleEpilogue se) {
  __shared__ float red[4][16][64];
  kslice_tile<MB, EPI, ST, 2>(X, W, out, M, N, K, kb_per_wave, se, blockIdx.x * 2, blockIdx.y, blockIdx.z, blockIdx.x, red);
}

// The same with tiles of two sizes in one launch, for matrices whose row blocks times K splits are three per compute
// unit (768 on this chip): n_big tiles of two row blocks per split come first in the grid, then n_small tiles of one.
// Two blocks fit a compute unit, and blocks are handed out in grid order to whatever unit has room: the first 256 land
// one per unit, the second 256 fill the remaining place of each, so every unit streams three row blocks -- the same
// bytes everywhere -- with two blocks resident, each hiding the other's start and end.  (Tiles of one size leave either
// 384 blocks, i.e. half of the units with twice the bytes of the rest, or 256 with nothing to overlap.)  Same K
// ranges, same order: same bits as every other variant.
// grid: x = splits * (n_big + n_small), z = M tile of 32*MB rows.
template <int MB, int EPI, int ST>
__global__ __launch_bounds__(256) void gemm_bf16_mixed_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                              void* __restrict__ out, int M, int N, int K, int kb_per_wave,
                                                              int n_big, int n_small, int splits, SampleEpilogue se) {
  static_assert(EPI != kEpiSample, "per-row-block epilogues only");
  __shared__ float red[4][16][64];
  const int id = blockIdx.x, all_big = splits * n_big;  // block-uniform
  if (id < all_big) {
    kslice_tile<MB, EPI, ST, 2>(X, W, out, M, N, K, kb_per_wave, se, (id % n_big) * 2, id / n_big, blockIdx.z, 0, red);
  } else {
    const int j = id - all_big;
    kslice_tile<MB, EPI, ST, 1>(X, W, out, M, N, K, kb_per_wave, se, 2 * n_big + j % n_small, j / n_small, blockIdx.z, 0, red);
  }
}

// Gate/up of one or two rows, with the residual sums and the RMSNorm before it.  A norm launch of its own takes 4 us, and the
// weights that follow wait for it.  Here every block forms the normalised rows itself: x and the split sums of the O projection are
// requested first, the weights of ST k blocks per wave right behind them, and while those travel the rows are summed, normalised and left in
// LDS as f16, from which the products take them.  No block waits for another (flags between blocks, written through:
// no faster than the two launches; with fences at device scope 14 us slower).  x is not changed: the split sums stay pending
// beside those of the down projection, for the next norm to add in the same order.
// Norm, gate/up and down over the weights of six layers, us: one row 54.0 -> 49.9, two rows 54.1 -> 51.9 (every block reads 80 KB per row
// from L2: more rows would pay more than the launch).  A layer of other shapes (hidden x ffn), one / two rows: 1024 x 512 32.8 -> 30.8 / 33.2 -> 32.3,
// 1024 x 3072 34.9 -> 32.8 / 35.0 -> 34.4, 2048 x 6144 44.7 -> 41.1 / 44.0 -> 42.3, 3072 x 8192 62.3 -> 59.6 / 60.3 -> 59.9, 4096 x 512 54.8 -> 50.7 / 54.2 -> 51.5.  Arithmetic of residual_norm_kernel and of the K-split kernels: same bits.
// grid: x = n_big tiles of two row blocks, then n_small of one (see gemm_bf16_mixed_kernel).
struct RowNorm {
  const float* x;
  const float* part;  // S <= kRowNormMaxS split sums, `stride` floats apart
  size_t stride;
  const uint16_t* gain;
  float eps;
  int S;
};
constexpr int kRowNormMaxS = 4, kRowNormPass = 1024, kRowNormMaxPass = 4;  // a pass: four elements per thread

template <int R, int ST, int RB>
__device__ __forceinline__ void row_tile(const RowNorm& rn, const u32x4_t* __restrict__ W, void* __restrict__ out, int M, int N,
                                        int K, int rb_first, float (&red)[4][16][64], u32x4_t* xs) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int KB = K >> 6, n = KB >> 2, passes = K / kRowNormPass;
  const u32x4_t* wr[RB];
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) wr[nb] = W + (size_t)(rb_first + nb) * KB * 256 + wave * 256 + lane;  // slot 4 b + wave: k block b of this wave's quarter
  u32x4_t f[ST][RB][4];
  auto load = [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) f[s][nb][t] = __builtin_nontemporal_load(wr[nb] + b * 1024 + t * 64);
  };
  auto barrier = []() __attribute__((always_inline)) {  // orders LDS alone: the weights stay in flight
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  float4 v[R][kRowNormMaxPass], p[R][kRowNormMaxS][kRowNormMaxPass];
  uint2 graw[kRowNormMaxPass];
#pragma unroll
  for (int q = 0; q < kRowNormMaxPass; ++q) {
    const int i0 = min(q, passes - 1) * kRowNormPass + threadIdx.x * 4;  // surplus passes repeat the last one and are dropped
    graw[q] = *(const uint2*)(rn.gain + i0);
#pragma unroll
    for (int r = 0; r < R; ++r) {
      const size_t at = (size_t)min(r, M - 1) * K + i0;
      v[r][q] = *(const float4*)(rn.x + at);
#pragma unroll
      for (int sp = 0; sp < kRowNormMaxS; ++sp) p[r][sp][q] = *(const float4*)(rn.part + min(sp, rn.S - 1) * rn.stride + at);
    }
  }
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int s = 0; s < ST; ++s) load(s, s);
  __builtin_amdgcn_sched_barrier(0);
  float* const ss = &red[0][0][0];
#pragma unroll
  for (int r = 0; r < R; ++r)
#pragma unroll
    for (int q = 0; q < kRowNormMaxPass; ++q) {
      float4 a = v[r][q];
#pragma unroll
      for (int sp = 0; sp < kRowNormMaxS; ++sp)
        if (sp < rn.S) {
          const float4 b = p[r][sp][q];
          a.x += b.x; a.y += b.y; a.z += b.z; a.w += b.w;
        }
      v[r][q] = a;
      const float sum = wave_sum((a.x * a.x + a.y * a.y) + (a.z * a.z + a.w * a.w));
      if (lane == 0) ss[(r * kRowNormMaxPass + q) * 4 + wave] = sum;
    }
  barrier();
#pragma unroll
  for (int r = 0; r < R; ++r) {
    float sum = 0.f;
    for (int w = 0; w < 4 * passes; ++w) sum += ss[r * kRowNormMaxPass * 4 + w];
    const float inv = 1.0f / sqrtf(sum / (float)K + rn.eps);
#pragma unroll
    for (int q = 0; q < kRowNormMaxPass; ++q) {
      if (q >= passes) break;
      const float4 a = v[r][q];
      const float4 g = make_float4(bf2f(graw[q].x & 0xffffu), bf2f(graw[q].x >> 16), bf2f(graw[q].y & 0xffffu), bf2f(graw[q].y >> 16));
      ((uint2*)xs)[r * (K >> 2) + q * (kRowNormPass / 4) + threadIdx.x] =
          make_uint2(pack2h(a.x * inv * g.x, a.y * inv * g.y), pack2h(a.z * inv * g.z, a.w * inv * g.w));
    }
  }
  barrier();
  f32x16_t acc[RB];
#pragma unroll
  for (int nb = 0; nb < RB; ++nb)
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[nb][r] = 0.f;
  const int col = lane & 31, hb = lane >> 5;
  const u32x4_t* const xl = xs + (size_t)min(col, R - 1) * (K >> 3) + wave * n * 8 + hb * 4;  // surplus columns repeat the last row, never stored
  auto multiply = [&](int s, int b) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const u32x4_t x = xl[b * 8 + t];
#pragma unroll
      for (int nb = 0; nb < RB; ++nb) acc[nb] = mfma_f16(f[s][nb][t], x, acc[nb]);
    }
  };
  int b = 0;
  for (; b + ST < n; b += ST) {  // n is a multiple of ST
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      multiply(s, b + s);
      __builtin_amdgcn_sched_barrier(0);
      load(s, b + s + ST);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < ST; ++s) multiply(s, b + s);
  float sum[RB][16];
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[nb][r];
    __syncthreads();
    if (wave == 0) {
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[nb][r] = ((red[0][r][lane] + red[1][r][lane]) + red[2][r][lane]) + red[3][r][lane];
    }
  }
  if (wave != 0 || col >= M) return;
#pragma unroll
  for (int nb = 0; nb < RB; ++nb) store_rowblock<kEpiSwiGLU>(sum[nb], col, hb, rb_first + nb, 0, M, N, out);
}

template <int R, int ST>
__global__ __launch_bounds__(256, 2) void norm_gate_up_kernel(RowNorm rn, const u32x4_t* __restrict__ W, void* __restrict__ out, int M,
                                                             int N, int K, int n_big) {
  __shared__ float red[4][16][64];
  __shared__ u32x4_t xs[R * kRowNormPass * kRowNormMaxPass / 8];
  const int id = blockIdx.x;  // block-uniform
  if (id < n_big) row_tile<R, ST, 2>(rn, W, out, M, N, K, id * 2, red, xs);
  else row_tile<R, ST, 1>(rn, W, out, M, N, K, n_big + id, red, xs);
}

// The K-split kernel with a 128-row weight tile (two 64-row pairs, four 32-row blocks per wave).  Every block reads
// the whole activation panel once, so halving the number of blocks halves that traffic; from about 48 rows on the
// panel reads of the 64-row tiling are as large as the weight stream itself and the launch is bound by what L2
// delivers.  Used where the halved grid still fills the chip.  Same K ranges per wave, same order: same bits.
template <int MB>
struct FragsW {
  u32x4_t a[4][4];
  u32x4_t b[MB][4];
};

template <int MB, int EPI, int ST>
__global__ __launch_bounds__(256, 1) void gemm_bf16_wide_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                              void* __restrict__ out, int M, int N, int K, int kb_per_wave,
                                                              SampleEpilogue se) {
  __shared__ float red[4][16][64];
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int KB = K >> 6;
  const int m_blk0 = blockIdx.z * MB;
  const int n_blocks_m = (M + 31) >> 5;
  const int n_tiles = EPI == kEpiSwiGLU ? (N >> 5) : (N >> 6);
  int tile[2], rb[4];
#pragma unroll
  for (int p = 0; p < 2; ++p) {
    tile[p] = min((int)blockIdx.x * 2 + p, n_tiles - 1);  // an odd tile count: the last block's second pair shadows its first
    rb[2 * p] = tile[p] * 2;
    rb[2 * p + 1] = tile[p] * 2 + 1;
  }
  const bool second_valid = (int)blockIdx.x * 2 + 1 < n_tiles;
  const u32x4_t* wp[4];
#pragma unroll
  for (int b = 0; b < 4; ++b) wp[b] = W + (size_t)rb[b] * KB * 256 + lane;
  const u32x4_t* xb[MB];
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    int b = m_blk0 + mb;
    if (b >= n_blocks_m) b = n_blocks_m - 1;  // clamp: surplus column blocks are computed but never stored
    xb[mb] = X + (size_t)b * KB * 256 + lane;
  }
  f32x16_t acc[4][MB];
#pragma unroll
  for (int b = 0; b < 4; ++b)
#pragma unroll
    for (int mb = 0; mb < MB; ++mb)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[b][mb][r] = 0.f;

  const int kw0 = blockIdx.y * 4 * kb_per_wave + wave - 4 * ((blockIdx.y * 4 + wave) * kb_per_wave);  // slot = kw0 + 4 kb
  auto load = [&](FragsW<MB>& f, int kb) __attribute__((always_inline)) {
    const int o = kb * 256, ow = (kw0 + 4 * kb) * 256;
#pragma unroll
    for (int t = 0; t < 4; ++t) {
#pragma unroll
      for (int b = 0; b < 4; ++b) f.a[b][t] = __builtin_nontemporal_load(wp[b] + ow + t * 64);
#pragma unroll
      for (int mb = 0; mb < MB; ++mb) f.b[mb][t] = xb[mb][o + t * 64];
    }
  };
  auto mma = [&](const FragsW<MB>& f) __attribute__((always_inline)) {
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
      for (int b = 0; b < 4; ++b) {
        const u32x4_t a = f.a[b][t];
#pragma unroll
        for (int mb = 0; mb < MB; ++mb) acc[b][mb] = mfma_f16(a, f.b[mb][t], acc[b][mb]);
      }
  };

  const int kb0 = (blockIdx.y * 4 + wave) * kb_per_wave;
  const int n = kb_per_wave;
  FragsW<MB> f[ST];
#pragma unroll
  for (int s = 0; s < ST; ++s) load(f[s], kb0 + s);  // the launcher guarantees ST <= n
  const int full = n / ST, rem = n - full * ST;
  int b = 0;
  for (int r = 0; r + 1 < full; ++r) {  // steady state: every buffer is refilled
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      mma(f[s]);
      __builtin_amdgcn_sched_barrier(0);
      load(f[s], kb0 + b + s + ST);
      __builtin_amdgcn_sched_barrier(0);
    }
    b += ST;
  }
  if (full > 0) {  // last full round: refill only what the remainder round will use
#pragma unroll
    for (int s = 0; s < ST; ++s) {
      mma(f[s]);
      __builtin_amdgcn_sched_barrier(0);
      if (s < rem) load(f[s], kb0 + b + s + ST);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int s = 0; s < ST; ++s)
    if (s < rem) mma(f[s]);

  // ---- add the four waves' accumulators (fixed order) and write: column block mb is finished by wave mb % 4 ----
  const int col = lane & 31, hb = lane >> 5;
#pragma unroll
  for (int mb = 0; mb < MB; ++mb) {
    float sum[4][16];
#pragma unroll
    for (int nb = 0; nb < 4; ++nb) {
      __syncthreads();
#pragma unroll
      for (int r = 0; r < 16; ++r) red[wave][r][lane] = acc[nb][mb][r];
      __syncthreads();
      if (wave == (mb & 3)) {
#pragma unroll
        for (int r = 0; r < 16; ++r)
          sum[nb][r] = ((red[0][r][lane] + red[1][r][lane]) + red[2][r][lane]) + red[3][r][lane];
      }
    }
    if (wave != (mb & 3)) continue;
    const int m = (m_blk0 + mb) * 32 + col;
    if (m >= M) continue;
#pragma unroll
    for (int p = 0; p < 2; ++p) {
      if (p == 1 && !second_valid) break;
      float pair[2][16];
#pragma unroll
      for (int nb = 0; nb < 2; ++nb)
#pragma unroll
        for (int r = 0; r < 16; ++r) pair[nb][r] = sum[2 * p + nb][r];
      store_block<EPI>(pair, m, hb, rb[2 * p], rb[2 * p + 1], blockIdx.y, M, N, out, se, tile[p]);
    }
  }
}

// Variant for 64 < M <= 256: the four waves take different batch-column blocks (MBW blocks of 32 each) instead of
// different K quarters, so a wave needs only 32*MBW accumulator columns and the block still streams W once (the
// four waves read the same weight tile at about the same time; only the first read leaves L2).  To keep a row's
// result bit-identical to the K-split variants, every wave still forms the four K-quarter sums separately and adds
// them in that order, ((q0 + q1) + q2) + q3, which needs two accumulator sets.
template <int MBW, int EPI, int ST>
__global__ __launch_bounds__(256) void gemm_bf16_cols_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                             void* __restrict__ out, int M, int N, int K, int kb_per_quarter,
                                                             SampleEpilogue se) {
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int KB = K >> 6;
  const int m_blk0 = (blockIdx.z * 4 + wave) * MBW;
  const int n_blocks_m = (M + 31) >> 5;
  if (m_blk0 >= n_blocks_m) return;  // this wave has no rows (no barriers below)

  int rb0, rb1;
  rb0 = blockIdx.x * 2;  // SwiGLU: the gate/up matrix is interleaved in 16-row groups, so this holds for it too
  rb1 = rb0 + 1;
  const u32x4_t* const wr[2] = {W + (size_t)rb0 * KB * 256, W + (size_t)rb1 * KB * 256};
  const u32x4_t* xb[MBW];
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    int b = m_blk0 + mb;
    if (b >= n_blocks_m) b = n_blocks_m - 1;
    xb[mb] = X + (size_t)b * KB * 256;
  }
  const int kb0 = blockIdx.y * 4 * kb_per_quarter;
  const int rounds = kb_per_quarter / ST;  // the launcher picks ST so that it divides kb_per_quarter
  Frags<MBW> f[ST];
  auto slot = [&](int kb) { return weight_kb_slot(kb, kb_per_quarter); };
#pragma unroll
  for (int s = 0; s < ST; ++s) load_frags<MBW, 2, false>(f[s], wr, xb, kb0 + s, slot(kb0 + s), lane);
  // One K quarter into a fresh accumulator.  The register ring keeps running across quarters: every block but the
  // last ST of the whole range re-issues its buffer for the block ST ahead.
  auto quarter = [&](f32x16_t (&a)[2][MBW], int q, bool last) __attribute__((always_inline)) {
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb)
#pragma unroll
        for (int r = 0; r < 16; ++r) a[nb][mb][r] = 0.f;
    const int base = kb0 + q * kb_per_quarter;
    const int refill_rounds = last ? rounds - 1 : rounds;
    for (int r = 0; r < refill_rounds; ++r) {
#pragma unroll
      for (int s = 0; s < ST; ++s) {
        mma_frags<MBW, 2>(f[s], a);
        __builtin_amdgcn_sched_barrier(0);
        load_frags<MBW, 2, false>(f[s], wr, xb, base + r * ST + s + ST, slot(base + r * ST + s + ST), lane);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (last) {
#pragma unroll
      for (int s = 0; s < ST; ++s) mma_frags<MBW, 2>(f[s], a);
    }
  };
  f32x16_t acc[2][MBW], other[2][MBW];
  quarter(acc, 0, false);
#pragma unroll
  for (int q = 1; q < 4; ++q) {
    quarter(other, q, q == 3);
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int mb = 0; mb < MBW; ++mb) acc[nb][mb] += other[nb][mb];
  }

  const int col = lane & 31, hb = lane >> 5;
#pragma unroll
  for (int mb = 0; mb < MBW; ++mb) {
    const int m = (m_blk0 + mb) * 32 + col;
    if (m >= M) continue;
    float sum[2][16];
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[nb][r] = acc[nb][mb][r];
    store_block<EPI>(sum, m, hb, rb0, rb1, blockIdx.y, M, N, out, se, blockIdx.x);
  }
}

// A full batch tile of eight waves (gate/up of 193..256 rows, QKV of 225..256): a 96-row weight tile (three row blocks) and all batch rows,
// where 128-row tiles would leave a quarter of the compute units without a block while 96-row tiles give every unit one.  (The same tile
// in gemm_bf16_tile_kernel: gate/up at 224 / 256 rows 60.1 / 62.9 us, here 59.3 / 59.8; QKV at 240 / 256 25.0 / 25.5, here 23.6 / 23.8.)  The first four waves stage
// row blocks 0 and 2, the other four row block 1; each half runs its own copy of the loop (same steps, one barrier
// per k block in both), so that no load in the pipeline is conditional.  Same K quarters, same order: same bits.
// grid: x = three row blocks, all of them whole, y = K split, K quarters of a multiple of four k blocks.  (Gate/up has one split; with
// a constant 0 in its place the compiler arranges the loop worse: 60.7 us at 256 rows instead of 59.8.)
template <int EPI>
__global__ __launch_bounds__(512, 1) void gemm_bf16_lds8r3_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                                void* __restrict__ out, int M, int N, int K,
                                                                int kb_per_quarter) {
  constexpr int RBN = 3, XS = 2;
  __shared__ u32x4_t wlds[4][RBN][256];  // four stages x three row blocks x 4 KiB
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int KB = K >> 6;
  const int n_blocks_m = (M + 31) >> 5;
  const int t256 = tid & 255;
  const int rb0 = blockIdx.x * RBN;
  const bool has_rows = wave < n_blocks_m;
  const u32x4_t* const xb = X + (size_t)min(wave, n_blocks_m - 1) * KB * 256 + lane;  // an idle wave shadows a valid block (never stored)
  const int n = 4 * kb_per_quarter;
  const int kb0 = blockIdx.y * n;
  auto kb_of = [&](int i) { return kb0 + (i < n ? i : n - 1); };  // clamped: no conditional loads in the pipeline
  f32x16_t acc[RBN];

  // NS = row blocks this half of the block stages: srb0 and, if there are two, srb1
  auto run = [&](auto ns_c, int srb0, int srb1) __attribute__((always_inline)) {
    constexpr int NS = decltype(ns_c)::value;
    const int srb[2] = {srb0, srb1};
    const u32x4_t* wp[NS];
#pragma unroll
    for (int b = 0; b < NS; ++b) wp[b] = W + (size_t)(rb0 + srb[b]) * KB * 256 + t256;
    // Weight k blocks are loaded strictly in order (the last one again once the range is exhausted); the slot of the
    // next one is kept as (block within its quarter, quarter) and stepped, without a division.
    int w_r = 0, w_q = 0;
    auto next_wslot = [&]() {
      const int off = (((int)blockIdx.y * kb_per_quarter + w_r) * 4 + w_q) * 256;
      if (w_r + 1 < kb_per_quarter) ++w_r;
      else if (w_q < 3) { w_r = 0; ++w_q; }
      return off;
    };
    u32x4_t wr[4][NS];   // weight registers: slot s holds a k block with index = s (mod 4)
    u32x4_t xr[XS][4];   // activation fragments: slot s holds a k block with index = s (mod XS)
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const int ow = next_wslot();
#pragma unroll
      for (int b = 0; b < NS; ++b) wr[s][b] = __builtin_nontemporal_load(wp[b] + ow);
    }
#pragma unroll
    for (int s = 0; s < XS; ++s)
#pragma unroll
      for (int t = 0; t < 4; ++t) xr[s][t] = xb[(size_t)kb_of(s) * 256 + t * 64];
    {
      const int ow = next_wslot();
#pragma unroll
      for (int b = 0; b < NS; ++b) {
        wlds[0][srb[b]][t256] = wr[0][b];
        wr[0][b] = __builtin_nontemporal_load(wp[b] + ow);
      }
    }
    auto iter = [&](f32x16_t (&a)[RBN], int i, auto jc) __attribute__((always_inline)) {
      constexpr int j = decltype(jc)::value, jn = (j + 1) & 3, jx = j % XS;
      const int ow = next_wslot();  // k block i + 5
#pragma unroll
      for (int b = 0; b < NS; ++b) {
        wlds[jn][srb[b]][t256] = wr[jn][b];
        wr[jn][b] = __builtin_nontemporal_load(wp[b] + ow);
      }
      // barrier that orders LDS traffic only (a full one would drain the global loads in flight)
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
      __builtin_amdgcn_s_barrier();
      __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int b = 0; b < RBN; ++b) a[b] = mfma_f16(wlds[j][b][t * 64 + lane], xr[jx][t], a[b]);
#pragma unroll
      for (int t = 0; t < 4; ++t) xr[jx][t] = xb[(size_t)kb_of(i + XS) * 256 + t * 64];
    };
    auto quarter = [&](f32x16_t (&a)[RBN], int q) __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < RBN; ++b)
#pragma unroll
        for (int r = 0; r < 16; ++r) a[b][r] = 0.f;
      for (int i = q * kb_per_quarter; i < (q + 1) * kb_per_quarter; i += 4) {
        iter(a, i, std::integral_constant<int, 0>{});
        iter(a, i + 1, std::integral_constant<int, 1>{});
        iter(a, i + 2, std::integral_constant<int, 2>{});
        iter(a, i + 3, std::integral_constant<int, 3>{});
      }
    };
    f32x16_t other[RBN];
    quarter(acc, 0);
    for (int q = 1; q < 4; ++q) {
      quarter(other, q);
#pragma unroll
      for (int b = 0; b < RBN; ++b) acc[b] += other[b];
    }
  };
  if (__builtin_amdgcn_readfirstlane(wave) < 4) run(std::integral_constant<int, 2>{}, 0, 2);
  else run(std::integral_constant<int, 1>{}, 1, 1);

  const int col = lane & 31, hb = lane >> 5, m = wave * 32 + col;
  if (!has_rows || m >= M) return;
#pragma unroll
  for (int b = 0; b < RBN; ++b) {
    float sum[16];
#pragma unroll
    for (int r = 0; r < 16; ++r) sum[r] = acc[b][r];
    store_rowblock<EPI>(sum, m, hb, rb0 + b, blockIdx.y, M, N, out);
  }
}

// More than 64 rows.  A block owns NB 32-row blocks of the weight matrix and NW * 32 batch rows, 32 per wave, over the K
// ranges of `splits` consecutive K splits.  The weight tile goes through LDS in three stages, one barrier per k block; the
// activation fragments come straight from L2.
//
// What bounds it.  At 1024 rows gate/up by itself spends 206 us with two resident blocks of four waves (128 x 128 each); without
// its activation loads 174, without its weight loads 150, without both and LDS 133, which is the matrix cores alone at
// the clock that their power leaves (operands of zeros: 176, 116, 95 and 94, so what a compute unit draws through its L1 is
// a bound of its own, at 70 GB/s per unit).  Both, the power and that rate, go by the bytes per product, hence (the launch by itself,
// without / with it):
//   - eight waves (128 x 256) where the batch fills them: 48 KB per k block instead of 64: 206 -> 190 us;
//   - weights that are read once (ONE: a single batch tile) pass through non-temporally: gate/up 41.0 -> 38.6 us at 72 rows;
//   - waves without batch rows carry weights and take part in the barriers, nothing else: gate/up at 301 rows 100 -> 84 us, down at
//     160 rows 40 -> 30; with four waves every other tile holds its rows in the other two
//     waves, so that two blocks on a unit do not leave the same matrix cores idle.  Not with a single batch tile of four
//     waves, where HBM is the bound and the second path only costs (128 rows: 42.9 -> 44.5).
// And one memory instruction behind every matrix instruction (a wave issues in order: a run of LDS writes or loads leaves
// its matrix core idle); the barrier does not wait for LDS reads in flight (a stage is rewritten one barrier after its last
// read); two waves per SIMD (256 registers), as two blocks of four or one of eight: four row blocks with running sums
// take 112 KB of LDS, so that one block of four waves is alone on a unit (O and down at 1024 rows).  Weights four k blocks
// ahead instead of two, or activations four ahead, gain nothing.
// The quarter sums keep a row's bits those of the K-split kernels: every K quarter in an accumulator of its own, added
// in order; then, where one block takes several K splits, the splits in order, kept in LDS between them.  So at more than
// 256 rows QKV, and at more than 512 O and down, leave no split partials: QKV writes its sum once, O and down
// add theirs to the residual stream themselves (kEpiResidual), in the order in which the norm kernel would.
// Kernel times in a step of the 8B shape (us), the staged kernels that it replaced -> now:
//   rows           72            128           160           192           301           512            640            768            1024
//   QKV       17.6 -> 15.7  18.8 -> 17.9  21.2 -> 20.5  21.6 -> 21.5  33.7 -> 33.5  38.4 -> 38.6   44.9 -> 45.3   59.8 -> 57.5   64.1 -> 61.2
//   O         14.6 -> 14.2  15.0 -> 15.4  18.4 -> 15.1  18.5 -> 15.7  25.0 -> 21.8  26.0 -> 25.5   36.8 -> 36.8   44.2 -> 43.9   47.0 -> 46.4
//   gate/up   41.8 -> 39.7  44.5 -> 44.9  56.5 -> 52.2  57.0 -> 55.3  86.9 -> 79.4 106.7 -> 107.3 141.8 -> 134.1 168.3 -> 157.5 202.7 -> 188.7
//   down      27.2 -> 26.8  29.1 -> 29.0  39.2 -> 32.0  39.1 -> 33.8  52.7 -> 44.0  55.7 -> 54.2   93.0 -> 93.1  112.1 -> 111.4 115.6 -> 115.7
__device__ __forceinline__ __amdgpu_buffer_rsrc_t buffer_of(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, bytes, 0x00020000);
}
__device__ __forceinline__ u32x4_t buffer_load16(__amdgpu_buffer_rsrc_t r, uint32_t voff, uint32_t soff) {
  return __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(r, voff, soff, 0));
}

constexpr int tile_sums_in_registers(int nb, int nw) { return nb == 3 && nw == 4 ? 1 : 0; }

template <int NB, int NW, int EPI, bool ONE>
__global__ __launch_bounds__(NW * 64, 2) void gemm_bf16_tile_kernel(const u32x4_t* __restrict__ X, const u32x4_t* __restrict__ W,
                                                              void* __restrict__ out, int M, int N, int K, int seg, int splits,
                                                              int n_tiles, int m_tiles, SampleEpilogue se) {
  static_assert(NB % 2 == 0 || EPI != kEpiSample, "the sampling epilogue works on pairs of row blocks");
  static_assert(NW == 4 || NW == 8, "four or eight waves");
  constexpr bool kIdleSkips = (!ONE || NW == 8) && EPI != kEpiResidual;
  constexpr int NF = NW == 8 ? NB / 2 : NB;          // 16-byte pieces of a k block of the tile per thread
  constexpr bool HALF = NW == 8 && (NB & 1) != 0;    // and one of 8 bytes
  constexpr int NC = NF + (HALF ? 1 : 0);
  constexpr bool kLate = NW == 4 && NB > 2 && !ONE;  // the last piece is staged early in the step after the others'
  constexpr int NE = kLate ? NC - 1 : NC;
  extern __shared__ u32x4_t smem[];  // three weight stages of NB x 4 KiB; then, with splits or a residual, the running sums
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int KB = splits * 4 * seg, kfirst = blockIdx.y * KB;  // k blocks of this block, the first one
  // Consecutive blocks go to the eight dies in turn: the batch tiles of one weight tile follow each other on one die.
  const int j = blockIdx.x >> 3;
  const int m_tile = j % m_tiles, n_tile = (j / m_tiles) * 8 + (blockIdx.x & 7);
  if (n_tile >= n_tiles) return;  // block-uniform
  const int n_rb = EPI == kEpiSwiGLU ? (N >> 4) : (N >> 5);
  const int n_mb = (M + 31) >> 5;
  const int rb0 = n_tile * NB;
  const int mb = m_tile * NW + (NW == 4 && kIdleSkips ? (wave + (n_tile & 1) * 2) & 3 : wave);
  const bool has_rows = mb < n_mb;  // idle waves carry weights and barriers; without kIdleSkips they also shadow the last rows
  const uint32_t row_bytes = (uint32_t)(K >> 6) * 4096;
  const auto wd = buffer_of((const char*)W + (size_t)rb0 * row_bytes, (uint32_t)min(NB, n_rb - rb0) * row_bytes);
  const int half = wave >> 2;  // eight waves: the first four stage row blocks 0 and 2, the others 1 and 3
  auto rb_of = [&](int c) __attribute__((always_inline)) { return NW == 8 ? 2 * c + half : c; };
  const auto xd = buffer_of((const char*)X + (size_t)min(mb, n_mb - 1) * row_bytes, row_bytes);
  const uint32_t wv = (tid & 255) * 16, xv = lane * 16, wv2 = tid * 8;
  int w_left = KB, w_r = 0, w_q = 0;
  uint32_t w_off = (uint32_t)kfirst * 4096;  // offset of the next weight k block to load (weight_kb_slot order)
  uint32_t w_row[NF + 1];
#pragma unroll
  for (int c = 0; c < NF; ++c) w_row[c] = (uint32_t)min(rb_of(c), n_rb - 1 - rb0) * row_bytes;
  w_row[NF] = (uint32_t)min(NB - 1, n_rb - 1 - rb0) * row_bytes;
  const int back = -((seg - 1) * 4 - 1) * 4096;
  auto next_w = [&]() __attribute__((always_inline)) {  // without branches; the last one again once the range is exhausted
    const bool wrap = ++w_r == seg;
    w_r = wrap ? 0 : w_r;
    w_q += wrap ? 1 : 0;
    const bool next = w_q == 4;
    w_q = next ? 0 : w_q;
    const int by = wrap ? (next ? 4096 : back) : 4 * 4096;
    w_off += --w_left > 0 ? by : 0;
  };
  constexpr int WS = 2, XS = 2;  // k blocks in registers beyond the stages in LDS
  typedef uint32_t u32x2_t __attribute__((ext_vector_type(2)));
  u32x4_t wr[WS][NF], xr[XS][4], fa[2][NB];  // weights on their way to LDS, activations, weight fragments of two phases
  u32x2_t wh[WS];
  auto load_x = [&](u32x4_t (&x)[4], int kb, int t) __attribute__((always_inline)) {
    x[t] = buffer_load16(xd, xv, (uint32_t)(kfirst + min(kb, KB - 1)) * 4096 + t * 1024);
  };
  // piece c of a k block of the tile: row block 2c + half, or half of the odd last one
  auto load_w = [&](int s, int c) __attribute__((always_inline)) {
    if (c < NF) wr[s][c] = __builtin_bit_cast(u32x4_t, __builtin_amdgcn_raw_buffer_load_b128(wd, wv, w_row[c] + w_off, ONE ? 2 : 0));
    else if (HALF) wh[s] = __builtin_bit_cast(u32x2_t, __builtin_amdgcn_raw_buffer_load_b64(wd, wv2, w_row[NF] + w_off, ONE ? 2 : 0));
  };
  auto put_w = [&](int stage, int s, int c) __attribute__((always_inline)) {
    if (c < NF) smem[(stage * NB + rb_of(c)) * 256 + (tid & 255)] = wr[s][c];
    else if (HALF) ((u32x2_t*)(smem + (stage * NB + NB - 1) * 256))[tid] = wh[s];
  };
  auto read = [&](u32x4_t (&f)[NB], int stage, int t, int b) __attribute__((always_inline)) { f[b] = smem[(stage * NB + b) * 256 + t * 64 + lane]; };
  auto barrier = []() __attribute__((always_inline)) {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
  };
  f32x16_t acc[NB], tot[NB];
#pragma unroll
  for (int s = 0; s < WS; ++s) {
#pragma unroll
    for (int c = 0; c < NC; ++c) load_w(s, c);
    next_w();
  }
#pragma unroll
  for (int s = 0; s < XS; ++s)
#pragma unroll
    for (int t = 0; t < 4; ++t) load_x(xr[s], s, t);
  // Running sums over the K splits, by lane: [row block][q][64 lanes] per wave in LDS; with three row blocks and four waves
  // the first one's stay in registers, which keeps two blocks on a compute unit.
  constexpr int UR = tile_sums_in_registers(NB, NW);
  f32x4_t* const usum = (f32x4_t*)(smem + 3 * NB * 256) + wave * (NB - UR) * 256 + lane;
  f32x4_t ureg[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) ureg[q] = (f32x4_t){0.f, 0.f, 0.f, 0.f};
  auto get_sum = [&](int b, int q) __attribute__((always_inline)) { return b < UR ? ureg[q] : usum[((b - UR) * 4 + q) * 64]; };
  auto set_sum = [&](int b, int q, f32x4_t v) __attribute__((always_inline)) {
    if (b < UR) ureg[q] = v;
    else usum[((b - UR) * 4 + q) * 64] = v;
  };
  const int col = lane & 31, hb = lane >> 5, m = mb * 32 + col;
  if (EPI == kEpiResidual) {
    const float* xo = (const float*)out + (size_t)min(m, M - 1) * N + 4 * hb;
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const f32x4_t v = *(const f32x4_t*)(xo + min(rb0 + b, n_rb - 1) * 32 + 8 * q);
        tot[b][4 * q] = v[0]; tot[b][4 * q + 1] = v[1]; tot[b][4 * q + 2] = v[2]; tot[b][4 * q + 3] = v[3];
      }
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        set_sum(b, q, (f32x4_t){tot[b][4 * q], tot[b][4 * q + 1], tot[b][4 * q + 2], tot[b][4 * q + 3]});
  }
  // stages 0 and 1 from registers 0 and 1; their registers take k blocks WS and WS + 1
#pragma unroll
  for (int s = 0; s < 2; ++s) {
    const int n = s == 0 ? NC : NE;
#pragma unroll
    for (int c = 0; c < n; ++c) put_w(s, s, c);
#pragma unroll
    for (int c = 0; c < n; ++c) load_w(s, c);
    if (s == 0 || !kLate) next_w();
  }
  barrier();
  if (kIdleSkips && !has_rows) {  // the steps below without products
    int rd = 1, wt = 2;
    for (int i = 0; i < KB; i += 2) {
      auto idle = [&](auto jc) __attribute__((always_inline)) {
        constexpr int J = decltype(jc)::value, jw = J, j1 = J ^ 1;
        if (kLate) {
          put_w(rd, j1, NC - 1);
          load_w(j1, NC - 1);
        }
        asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory");
        if (kLate) next_w();
#pragma unroll
        for (int c = 0; c < NE; ++c) put_w(wt, jw, c);
#pragma unroll
        for (int c = 0; c < NE; ++c) load_w(jw, c);
        if (!kLate) next_w();
        rd = wt;
        wt = wt == 2 ? 0 : wt + 1;
      };
      idle(std::integral_constant<int, 0>{});
      idle(std::integral_constant<int, 1>{});
    }
    return;
  }
#pragma unroll
  for (int t = 0; t < 2; ++t)
#pragma unroll
    for (int b = 0; b < NB; ++b) read(fa[t], 0, t, b);
  int cur = 0, rd = 1, wt = 2;  // LDS stages of k blocks i, i + 1 and i + 2
  auto step = [&](int i, auto jc, auto fc) __attribute__((always_inline)) {
    constexpr int J = decltype(jc)::value, jx = J & 1, jw = J & 1, j1 = jw ^ 1;  // k block i + 2 waits in register slot jw
    constexpr bool first = decltype(fc)::value;
    auto phase = [&](auto pc) __attribute__((always_inline)) {
      constexpr int P = decltype(pc)::value;
#pragma unroll
      for (int b = 0; b < NB; ++b) {
        f32x16_t c;
        if constexpr (first && P == 0) {
#pragma unroll
          for (int r = 0; r < 16; ++r) c[r] = 0.f;
        } else {
          c = acc[b];
        }
        acc[b] = mfma_f16(fa[P & 1][b], xr[jx][P], c);
        read(fa[P & 1], P < 2 ? cur : rd, (P + 2) & 3, b);  // past the last k block: a stage nobody needs, never used
        // one more memory instruction behind each matrix instruction
        if constexpr (kLate) {
          if (P == 0 && b == 0) put_w(rd, j1, NC - 1);
          if (P == 0 && b == 1) load_x(xr[jx ^ 1], i + 1, 3);
          if (P == 0 && b == 2 && NB == 4) load_w(j1, 2);
          if (P == 1 && b == 0) load_w(j1, NC - 1);
          if (P == 1 && b == 1) load_x(xr[jx], i + 2, 0);
          if (P == 2 && b == 0) put_w(wt, jw, 0);
          if (P == 2 && b == 1) load_x(xr[jx], i + 2, 1);
          if (P == 2 && b == 2 && NB == 4) put_w(wt, jw, 1);
          if (P == 3 && b == 0) put_w(wt, jw, NC - 2);
          if (P == 3 && b == 1) load_x(xr[jx], i + 2, 2);
          if (P == 3 && b == NB - 1) {
            next_w();
            load_w(jw, 0);
            load_w(jw, 1);
          }
        } else {
          if (b == NB - 1) load_x(xr[jx], i + 2, P);
          if (P >= 2) {
            constexpr int c0 = P - 2, c1 = P;
            if (c0 < NC && b == 0) put_w(wt, jw, c0);
            if (c0 < NC && b == 1) load_w(jw, c0);
            if (c1 < NC && b == NB / 2) put_w(wt, jw, c1);
            if (c1 < NC && b == NB - 1) load_w(jw, c1);
          }
          if (P == 3 && b == NB - 1) next_w();
        }
        __builtin_amdgcn_sched_barrier(0);
      }
    };
    phase(std::integral_constant<int, 0>{});
    phase(std::integral_constant<int, 1>{});
    // LDS operations of a wave finish in order: with at most phase 1's reads outstanding, the stage of k block i + 1 is
    // complete and all reads of k block i - 1, whose stage is written next, are done.
    asm volatile("s_waitcnt lgkmcnt(%0)\n\ts_barrier" :: "n"(NB) : "memory");
    phase(std::integral_constant<int, 2>{});
    phase(std::integral_constant<int, 3>{});
    const int c = cur;
    cur = rd;
    rd = wt;
    wt = c;
  };
  auto steps4 = [&](int i, auto fc) __attribute__((always_inline)) {
    step(i, std::integral_constant<int, 0>{}, fc);
    step(i + 1, std::integral_constant<int, 1>{}, std::false_type{});
    step(i + 2, std::integral_constant<int, 2>{}, std::false_type{});
    step(i + 3, std::integral_constant<int, 3>{}, std::false_type{});
  };
  int i = 0;
  for (int sp = 0; sp < splits; ++sp) {
#pragma unroll
    for (int b = 0; b < NB; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) tot[b][r] = -0.0f;  // -0 + x is x, bit for bit
    for (int q = 0; q < 4; ++q) {
      steps4(i, std::true_type{});
      for (int e = i + seg, k = i + 4; k < e; k += 4) steps4(k, std::false_type{});
      i += seg;
#pragma unroll
      for (int b = 0; b < NB; ++b) tot[b] += acc[b];
    }
    if (EPI == kEpiResidual || (EPI == kEpiPartial && splits > 1)) {
#pragma unroll
      for (int b = 0; b < NB; ++b)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          f32x4_t v = {tot[b][4 * q], tot[b][4 * q + 1], tot[b][4 * q + 2], tot[b][4 * q + 3]};
          if (EPI == kEpiResidual || sp > 0) v = get_sum(b, q) + v;
          if (sp + 1 < splits) set_sum(b, q, v);
          else { tot[b][4 * q] = v[0]; tot[b][4 * q + 1] = v[1]; tot[b][4 * q + 2] = v[2]; tot[b][4 * q + 3] = v[3]; }
        }
    }
  }
  if (!has_rows || m >= M) return;
  if constexpr (EPI == kEpiSample) {
#pragma unroll
    for (int b = 0; b < NB; b += 2) {
      float sum[2][16];
#pragma unroll
      for (int r = 0; r < 16; ++r) { sum[0][r] = tot[b][r]; sum[1][r] = tot[b + 1][r]; }
      if (rb0 + b < n_rb) store_block<EPI>(sum, m, hb, rb0 + b, rb0 + b + 1, 0, M, N, out, se, (rb0 + b) >> 1);
    }
  } else {
#pragma unroll
    for (int b = 0; b < NB; ++b) {
      float sum[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) sum[r] = tot[b][r];
      if (rb0 + b < n_rb) store_rowblock<EPI == kEpiResidual ? kEpiPartial : EPI>(sum, m, hb, rb0 + b, blockIdx.y, M, N, out);
    }
  }
}

template <int MB, int ST>
void launch_mb(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
               const SampleEpilogue& se) {
  GemmPlan p = gemm_plan(N, K, epi, allow_split);
  const int m_tiles = (M + 32 * MB - 1) / (32 * MB);
  if (epi == kEpiSwiGLU) {
    dim3 grid(N >> 5, 1, m_tiles);
    gemm_bf16_kernel<MB, kEpiSwiGLU, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  } else if (epi == kEpiSample) {
    dim3 grid(N >> 6, 1, m_tiles);
    gemm_bf16_kernel<MB, kEpiSample, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  } else {
    dim3 grid(N >> 6, p.splits, m_tiles);
    gemm_bf16_kernel<MB, kEpiPartial, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  }
}

template <int MB, int ST>
void launch_wide(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
                 const SampleEpilogue& se) {
  GemmPlan p = gemm_plan(N, K, epi, allow_split);  // same K split as the narrow tiling: bit-identical results
  const int m_tiles = (M + 32 * MB - 1) / (32 * MB);
  const int tiles = epi == kEpiSwiGLU ? (N >> 5) : (N >> 6);
  dim3 grid((tiles + 1) / 2, epi == kEpiPartial ? p.splits : 1, m_tiles);
  if (epi == kEpiSwiGLU)
    gemm_bf16_wide_kernel<MB, kEpiSwiGLU, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  else if (epi == kEpiSample)
    gemm_bf16_wide_kernel<MB, kEpiSample, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  else
    gemm_bf16_wide_kernel<MB, kEpiPartial, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
}

template <int MB, int ST>
void launch_mixed(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
                  const SampleEpilogue& se) {
  const GemmPlan p = gemm_plan(N, K, epi, allow_split);  // same K split as the other variants: bit-identical results
  const int row_blocks = (epi == kEpiSwiGLU ? 2 * N : N) >> 5, third = row_blocks / 3;
  const int m_tiles = (M + 32 * MB - 1) / (32 * MB);
  dim3 grid(p.splits * 2 * third, 1, m_tiles);
  if (epi == kEpiSwiGLU)
    gemm_bf16_mixed_kernel<MB, kEpiSwiGLU, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K,
                                                                    p.kb_per_wave, third, third, p.splits, se);
  else
    gemm_bf16_mixed_kernel<MB, kEpiPartial, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K,
                                                                     p.kb_per_wave, third, third, p.splits, se);
}

template <int NB, int NW, bool ONE>
void launch_tile(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
                 const SampleEpilogue& se) {
  const GemmPlan p = gemm_plan(N, K, epi == kEpiResidual ? kEpiPartial : epi, allow_split);  // same K split as the other variants: bit-identical results
  const bool whole = gemm_whole_k(M, N, K, epi, allow_split);
  const int n_rb = epi == kEpiSwiGLU ? (N >> 4) : (N >> 5);
  const int n_tiles = (n_rb + NB - 1) / NB, m_tiles = (M + 32 * NW - 1) / (32 * NW), splits = whole ? p.splits : 1;
  dim3 grid((n_tiles + 7) / 8 * 8 * m_tiles, whole ? 1 : p.splits);
  const bool sums = splits > 1 || epi == kEpiResidual;
  const size_t lds = (size_t)NB * 3 * 4096 + (sums ? (size_t)(NB - tile_sums_in_registers(NB, NW)) * NW * 4096 : 0);
#define RL_TILE(E) gemm_bf16_tile_kernel<NB, NW, E, ONE><<<grid, NW * 64, lds, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, splits, n_tiles, m_tiles, se)
  if (epi == kEpiSwiGLU) RL_TILE(kEpiSwiGLU);
  else if (epi == kEpiResidual) { if constexpr (!ONE && NB > 2) RL_TILE(kEpiResidual); }
  else if (epi == kEpiSample) { if constexpr (NB % 2 == 0) RL_TILE(kEpiSample); }
  else RL_TILE(kEpiPartial);
#undef RL_TILE
}

}  // namespace

int gemm_bf16_partials(int M, int N, int K) { return gemm_whole_k(M, N, K, kEpiPartial, true) ? 1 : gemm_bf16_splits(N, K, kEpiPartial); }
bool gemm_bf16_adds_residual(int M, int N, int K) { return gemm_whole_k(M, N, K, kEpiResidual, true); }
int gemm_bf16_splits(int N, int K, int epi) { return gemm_plan(N, K, epi, true).splits; }
int gemm_bf16_weight_segment(int N, int K, bool split_k) { return gemm_plan(N, K, kEpiPartial, split_k).kb_per_wave; }

// Whole k blocks per wave and pass: hidden a multiple of 1024; the K quarters hold at least the four k blocks of the ring.
bool norm_gate_up_takes(int M, int H, int S) { return M <= 2 && H % kRowNormPass == 0 && H <= kRowNormPass * kRowNormMaxPass && S >= 1 && S <= kRowNormMaxS; }

void launch_norm_gate_up(hipStream_t s, const float* x, const float* part, int S, const void* gain, float eps, const void* W, void* out,
                         int M, int F, int H) {
  const RowNorm rn = {x, part, (size_t)M * H, (const uint16_t*)gain, eps, S};
  const int tiles = F >> 4;  // row blocks of the interleaved matrix
  const bool mixed = gemm_mixed_fits(F, H, kEpiSwiGLU, true);
  const int n_big = mixed ? tiles / 3 : tiles / 2, blocks = mixed ? 2 * n_big : n_big;
  if (M == 1) norm_gate_up_kernel<1, 4><<<blocks, 256, 0, s>>>(rn, (const u32x4_t*)W, out, M, F, H, n_big);
  else norm_gate_up_kernel<2, 2><<<blocks, 256, 0, s>>>(rn, (const u32x4_t*)W, out, M, F, H, n_big);
}

template <int MB>
void launch_st(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
               int stages, const SampleEpilogue& se) {
  const int n = gemm_plan(N, K, epi, allow_split).kb_per_wave;
  if (stages > n) stages = n;  // the kernel's prologue fills all of its buffers unconditionally
  switch (stages) {
    case 1: launch_mb<MB, 1>(s, X, W, out, M, N, K, epi, allow_split, se); break;
    case 2: launch_mb<MB, 2>(s, X, W, out, M, N, K, epi, allow_split, se); break;
    case 3: launch_mb<MB, 3>(s, X, W, out, M, N, K, epi, allow_split, se); break;
    default: launch_mb<MB, 4>(s, X, W, out, M, N, K, epi, allow_split, se); break;
  }
}

template <int MBW, int ST>
void launch_cols_st(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
                    const SampleEpilogue& se) {
  GemmPlan p = gemm_plan(N, K, epi, allow_split);  // same K split as the other variants: bit-identical results
  const int m_tiles = (M + 128 * MBW - 1) / (128 * MBW);
  if (epi == kEpiSwiGLU) {
    dim3 grid(N >> 5, 1, m_tiles);
    gemm_bf16_cols_kernel<MBW, kEpiSwiGLU, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  } else if (epi == kEpiSample) {
    dim3 grid(N >> 6, 1, m_tiles);
    gemm_bf16_cols_kernel<MBW, kEpiSample, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  } else {
    dim3 grid(N >> 6, p.splits, m_tiles);
    gemm_bf16_cols_kernel<MBW, kEpiPartial, ST><<<grid, 256, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave, se);
  }
}

// More than 64 rows.
template <int MBW>
void launch_cols(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi, bool allow_split,
                 const SampleEpilogue& se) {
  const GemmPlan p = gemm_plan(N, K, epi == kEpiResidual ? kEpiPartial : epi, allow_split);
  if (p.kb_per_wave % 4 == 0) {  // weight tiles shared through LDS
    const GemmTile t = gemm_tile(M, N, K, epi, allow_split);
    // A full batch tile on 96-row weight tiles.  The lines: gate/up at 192 rows, where two waves of the tile kernel rest, 56.7 us there and 59.0
    // here, at 224 60.1 and 59.3; QKV at 224 rows 23.7 and 23.4, at 256 25.5 and 23.8.  In eight splits the tile kernel stays ahead (down of 3072 x
    // 8192 at 240 rows 25.2 and 25.9).
    if (t.nb == 3 && t.nw == 8 && M <= 256 && (epi == kEpiSwiGLU ? M > 192 : M > 224 && p.splits <= 4)) {
      const dim3 grid((epi == kEpiSwiGLU ? N >> 4 : N >> 5) / 3, p.splits);
      if (epi == kEpiSwiGLU) gemm_bf16_lds8r3_kernel<kEpiSwiGLU><<<grid, 512, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave);
      else gemm_bf16_lds8r3_kernel<kEpiPartial><<<grid, 512, 0, s>>>((const u32x4_t*)X, (const u32x4_t*)W, out, M, N, K, p.kb_per_wave);
      return;
    }
    const bool one = M <= 32 * t.nw;  // a single batch tile
#define RL_PICK(NB, NW) \
  if (t.nb == NB && t.nw == NW) { \
    if (one) launch_tile<NB, NW, true>(s, X, W, out, M, N, K, epi, allow_split, se); \
    else launch_tile<NB, NW, false>(s, X, W, out, M, N, K, epi, allow_split, se); \
    return; \
  }
    RL_PICK(4, 4)
    RL_PICK(3, 4)
    RL_PICK(2, 4)
    RL_PICK(4, 8)
    RL_PICK(3, 8)
#undef RL_PICK
  }
  // two buffers in flight per wave when the quarter length allows it
  if (p.kb_per_wave % 2 == 0) launch_cols_st<MBW, 2>(s, X, W, out, M, N, K, epi, allow_split, se);
  else launch_cols_st<MBW, 1>(s, X, W, out, M, N, K, epi, allow_split, se);
}

// Requirements (checked at model init): K % 256 == 0, N % 64 == 0 (N % 32 for SwiGLU).
void launch_gemm_bf16(hipStream_t s, const void* X, const void* W, void* out, int M, int N, int K, int epi,
                      bool allow_split, const SampleEpilogue* se) {
  static const SampleEpilogue none{};
  const SampleEpilogue& e = se ? *se : none;
  if (epi == kEpiSample) allow_split = false;
  // 128-row tiles for the K-split projections whose halved grid still fills the chip (QKV at the 8B shape: 16 -> 15 us
  // at 32 rows, 20.5 -> 17.8 us at 64); measured a loss for gate/up and the output projection, which keep 64-row tiles.
  const bool wide = epi == kEpiPartial && gemm_plan(N, K, epi, allow_split).splits > 1 &&
                    gemm_wide_blocks(N, K, epi, allow_split) >= 192 && gemm_plan(N, K, epi, allow_split).kb_per_wave >= 2;
  const bool mixed = gemm_mixed_fits(N, K, epi, allow_split);
  const int kbw = gemm_plan(N, K, epi, allow_split).kb_per_wave;
  if (M <= 32 && mixed && kbw >= 4) launch_mixed<1, 4>(s, X, W, out, M, N, K, epi, allow_split, e);
  else if (M <= 64 && M > 32 && mixed && kbw >= 2) launch_mixed<2, 2>(s, X, W, out, M, N, K, epi, allow_split, e);
  else if (M <= 32 && wide) launch_wide<1, 2>(s, X, W, out, M, N, K, epi, allow_split, e);
  else if (M <= 32) launch_st<1>(s, X, W, out, M, N, K, epi, allow_split, 4, e);
  else if (M <= 64 && wide) launch_wide<2, 2>(s, X, W, out, M, N, K, epi, allow_split, e);
  else if (M <= 64) launch_st<2>(s, X, W, out, M, N, K, epi, allow_split, 2, e);
  else if (M <= 128) launch_cols<1>(s, X, W, out, M, N, K, epi, allow_split, e);
  else launch_cols<2>(s, X, W, out, M, N, K, epi, allow_split, e);
}

}  // namespace rl
