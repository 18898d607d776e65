// First kernel of a call, residual + RMSNorm, per-head norm + rotary + KV append, KV import, weight packing.
// These move little data per step; they are written for few launches and simple indexing.
#include <algorithm>

#include "device_utils.h"
#include "kernels.h"
#include "rope_device.h"

namespace rl {

// ------------------------------------------------------------------------------------------------
// First kernel of a call: the call's metadata slot (rows, tokens, attention plan) moves from pinned host memory to the
// device, new pages are entered in the block table, and the rows enter the residual stream (from the embedding table or
// from the caller's buffer) and, in bf16 models, the first layer's RMSNorm.
//
// Each of these used to be a launch of its own: a copy of the slot (a blit kernel, 2 to 4 us), the table update, the
// copy of the caller's rows and the norm are a chain in which every link costs a launch and at least one round trip to
// memory.  Here a few leading blocks read the slot while the others work on their rows.  Together with the last copy (the
// sums behind the last layer go straight to the caller's buffer) and one event per twelve calls instead of per call: one
// layer on one row 109.9 -> 99.5 us, on 64 rows 205.0 -> 194.0.
// ------------------------------------------------------------------------------------------------
__host__ __device__ inline int slot_units(const SlotUpload& u) {
  int n = u.n_rows;
  for (int k = 0; k < kSlotRegions; ++k) n += u.n[k];
  return n;
}

__device__ __forceinline__ void upload_slot(const SlotUpload& u, int first, int stride) {
  const int total = slot_units(u);
  for (int i = first; i < total; i += stride) {
    int at = i, left = i - u.n_rows;
    if (left >= 0) {
#pragma unroll
      for (int k = 0; k < kSlotRegions; ++k) {
        if (left >= 0 && left < u.n[k]) at = u.at[k] + left;
        left -= u.n[k];
      }
    }
    const uint4 v = u.src[at];
    u.dst[at] = v;
    // A row at the first position of a page names that page (RowMeta: seq, pos, page): its block-table entry.  Every page
    // a sequence grows into gets its first row before any row reads it, so this is all the table needs.
    if (i < u.n_rows && u.block_table && (v.y & (kPageTokens - 1)) == 0) u.block_table[(size_t)v.x * u.max_blocks + (v.y >> 4)] = (int32_t)v.z;
  }
}

// Tokens of rows r .. r + R - 1 (past the last row: its token again): each is read by one lane per block, because the tokens of
// a prompt (and the rows of a step that feeds itself) lie in host memory.
template <int R>
__device__ __forceinline__ void fetch_tokens(const RowSource& in, int r, int M, int (&shared)[R]) {
  if (threadIdx.x < R) {
    const int i = min(r + (int)threadIdx.x, M - 1);
    const int fed = in.tokens != nullptr ? in.tokens[i] : in.last_tok[in.rows[i].seq];
    shared[threadIdx.x] = min(max(fed, 0), in.V - 1);  // ids come from device memory the host cannot inspect
  }
  __syncthreads();
}

template <typename T>
__global__ __launch_bounds__(256) void entry_rows_kernel(RowSource in, SlotUpload up, int up_blocks, float* __restrict__ x, int H) {
  __shared__ int token[1];
  if ((int)blockIdx.x < up_blocks) {
    upload_slot(up, blockIdx.x * 256 + threadIdx.x, up_blocks * 256);
    return;
  }
  const int r = blockIdx.x - up_blocks;
  if (in.from_table) fetch_tokens(in, r, r + 1, token);
  const size_t base = (size_t)(in.from_table ? token[0] : r) * H;
  for (int i = threadIdx.x; i < H; i += 256) x[(size_t)r * H + i] = load_as_float((const T*)in.src, base + i);
}

// ------------------------------------------------------------------------------------------------
// Residual update + RMSNorm.  One block per row, one float4 per thread and pass (H/4 threads, at most 1024), so
// that the few dependent memory round trips of this latency-bound step are as short as possible.  The split
// partials of the preceding projection are summed in a fixed order, so results do not depend on the batch.  bf16 models
// only: fp32 projections normalise their rows and add to the residual stream themselves.
// ------------------------------------------------------------------------------------------------
// SRC 0: x = xi + split sums, 3: the same with row r from row r / group;  1: the rows of a call from the caller's fp32 buffer;  2: from the embedding table (bf16).
// 1 and 2 are the first kernel of a call: x is always written, and leading blocks move the metadata slot.
// xo may be xi.  gain: H bf16 gains; without a norm (has_gain = 0) any readable H-element array.
// R: rows per block.  A block of 1024 threads spends its time on one round trip and a barrier, and two blocks fill a compute
// unit: beyond 512 rows, two rows per block keep it at one round of blocks (1024 rows 11.3 -> 8.3 us, from the table 18.3 -> 13.0;
// 513 rows 7.2 -> 6.0 and 11.8 -> 9.9; 512 rows 11.2 -> 10.7 with four split sums to add, and 9.9 -> 10.0).  A row's bits do not
// depend on R.
template <int SRC, int R>
__global__ __launch_bounds__(1024) void residual_norm_kernel(const float* xi, float* xo, const float* __restrict__ part,
                                                             int S, size_t split_stride, const void* __restrict__ gain,
                                                             int has_gain, void* __restrict__ h_out,
                                                             float* __restrict__ capture, int H, float eps, RowSource in,
                                                             SlotUpload up, int up_blocks, int group, int M) {
  __shared__ float red[R][16];
  __shared__ int token[R];
  const int nthr = blockDim.x;
  constexpr bool kEntry = SRC == 1 || SRC == 2;
  if (kEntry && (int)blockIdx.x < up_blocks) {
    upload_slot(up, blockIdx.x * nthr + threadIdx.x, up_blocks * nthr);
    return;
  }
  static_assert(R == 1 || SRC != 3, "a group's rows have blocks of their own");
  const int r0 = (kEntry ? (int)blockIdx.x - up_blocks : (int)blockIdx.x) * R;
  constexpr int kMaxPass = 2;  // H <= 1024 threads * 4 * kMaxPass, checked by the host
  float4 keep[R][kMaxPass];
  float ss[R];
  // Gains are requested together with the data, as stored (two words per thread), and first touched after the
  // sums: converting them here would make the compiler wait for them before it even asks for the data.
  uint2 graw[kMaxPass];
#pragma unroll
  for (int pass = 0; pass < kMaxPass; ++pass) {
    const int i0 = (pass * nthr + threadIdx.x) * 4;
    const int ig = i0 < H ? i0 : 0;  // unconditional loads (a branch here costs a wait); `gain` is always readable
    graw[pass] = *(const uint2*)((const uint16_t*)gain + ig);
  }
  if (SRC == 2) fetch_tokens(in, r0, M, token);
#pragma unroll
  for (int pass = 0; pass < kMaxPass; ++pass) {
    const int i0 = (pass * nthr + threadIdx.x) * 4;
#pragma unroll
    for (int k = 0; k < R; ++k) keep[k][pass] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (i0 < H) {
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int ri = SRC == 3 ? r0 / group : min(r0 + k, M - 1);
        if (SRC == 2) {
          const uint2 e = *(const uint2*)((const uint16_t*)in.src + (size_t)token[k] * H + i0);
          keep[k][pass] = make_float4(bf2f(e.x & 0xffffu), bf2f(e.x >> 16), bf2f(e.y & 0xffffu), bf2f(e.y >> 16));
        } else {
          keep[k][pass] = *(const float4*)(xi + (size_t)ri * H + i0);
        }
      }
#pragma unroll
      for (int k = 0; k < R; ++k) {
        const int ri = SRC == 3 ? r0 / group : min(r0 + k, M - 1);
        float4 v = keep[k][pass];
#pragma unroll 4
        for (int sp = 0; sp < S; ++sp) {
          const float4 p = *(const float4*)(part + sp * split_stride + (size_t)ri * H + i0);
          v.x += p.x; v.y += p.y; v.z += p.z; v.w += p.w;
        }
        keep[k][pass] = v;
        if (R > 1 && r0 + k >= M) continue;
        if (kEntry || S > 0) *(float4*)(xo + (size_t)(r0 + k) * H + i0) = v;
        if (capture) *(float4*)(capture + (size_t)(r0 + k) * H + i0) = v;
      }
    }
  }
  if (!has_gain) return;
#pragma unroll
  for (int pass = 0; pass < kMaxPass; ++pass)
    asm volatile("" : "+v"(graw[pass].x), "+v"(graw[pass].y));
#pragma unroll
  for (int k = 0; k < R; ++k) {
    ss[k] = 0.f;
#pragma unroll
    for (int pass = 0; pass < kMaxPass; ++pass) {
      const float4 v = keep[k][pass];
      ss[k] += (v.x * v.x + v.y * v.y) + (v.z * v.z + v.w * v.w);
    }
    ss[k] = wave_sum(ss[k]);
    if ((threadIdx.x & 63) == 0) red[k][threadIdx.x >> 6] = ss[k];
  }
  __syncthreads();
#pragma unroll
  for (int k = 0; k < R; ++k) {
    if (R > 1 && r0 + k >= M) continue;
    float sum = 0.f;
    for (int w = 0; w < (nthr >> 6); ++w) sum += red[k][w];
    const float inv = 1.0f / sqrtf(sum / (float)H + eps);
#pragma unroll
    for (int pass = 0; pass < kMaxPass; ++pass) {
      const int i0 = (pass * nthr + threadIdx.x) * 4;
      if (i0 >= H) continue;
      const float4 v = keep[k][pass];
      const float4 g = make_float4(bf2f(graw[pass].x & 0xffffu), bf2f(graw[pass].x >> 16), bf2f(graw[pass].y & 0xffffu), bf2f(graw[pass].y >> 16));
      *(uint2*)((uint16_t*)h_out + frag_offset(r0 + k, i0, H >> 6)) =
          make_uint2(pack2h(v.x * inv * g.x, v.y * inv * g.y), pack2h(v.z * inv * g.z, v.w * inv * g.w));
    }
  }
}

static int norm_threads(int H) { return std::min(((H / 4 + 63) / 64) * 64, 1024); }

void launch_residual_norm(hipStream_t s, const float* x_in, float* x_out, const float* part, int S, const void* gain,
                          void* h_out, float* capture, int M, int H, float eps, int group) {
  const int has_gain = gain != nullptr;
  const void* g = has_gain ? gain : x_in;  // read and ignored without a norm
  const size_t stride = (size_t)(M / group) * H;
  if (group > 1)
    residual_norm_kernel<3, 1><<<M, norm_threads(H), 0, s>>>(x_in, x_out, part, S, stride, g, has_gain, h_out, capture, H, eps, RowSource{}, SlotUpload{}, 0, group, M);
  else if (M > 512)
    residual_norm_kernel<0, 2><<<(M + 1) / 2, norm_threads(H), 0, s>>>(x_in, x_out, part, S, stride, g, has_gain, h_out, capture, H, eps, RowSource{}, SlotUpload{}, 0, 1, M);
  else
    residual_norm_kernel<0, 1><<<M, norm_threads(H), 0, s>>>(x_in, x_out, part, S, stride, g, has_gain, h_out, capture, H, eps, RowSource{}, SlotUpload{}, 0, 1, M);
}

void launch_entry(hipStream_t s, int dtype, const RowSource& in, const SlotUpload& up, float* x, const void* gain, void* h_out,
                  float* capture, int M, int H, float eps) {
  const int words = slot_units(up);
  // The fused kernel reads 16 bytes of an fp32 row or 8 of a table row at a time; the caller's buffer or a table that is
  // not aligned to that goes element by element, and a norm of its own follows.
  const bool fused = dtype == kBF16 && (uintptr_t)in.src % (in.from_table ? 8 : 16) == 0;
  if (!fused) {
    const int up_blocks = (words + 255) / 256;
    if (in.from_table && dtype == kBF16) entry_rows_kernel<uint16_t><<<M + up_blocks, 256, 0, s>>>(in, up, up_blocks, x, H);
    else entry_rows_kernel<float><<<M + up_blocks, 256, 0, s>>>(in, up, up_blocks, x, H);
    if (dtype == kBF16) launch_residual_norm(s, x, x, nullptr, 0, gain, h_out, capture, M, H, eps);
    return;
  }
  const int threads = norm_threads(H), up_blocks = (words + threads - 1) / threads;
  if (!in.from_table)
    residual_norm_kernel<1, 1><<<M + up_blocks, threads, 0, s>>>((const float*)in.src, x, nullptr, 0, 0, gain, 1, h_out, capture, H, eps, in, up, up_blocks, 1, M);
  else if (M > 512)
    residual_norm_kernel<2, 2><<<(M + 1) / 2 + up_blocks, threads, 0, s>>>(nullptr, x, nullptr, 0, 0, gain, 1, h_out, capture, H, eps, in, up, up_blocks, 1, M);
  else
    residual_norm_kernel<2, 1><<<M + up_blocks, threads, 0, s>>>(nullptr, x, nullptr, 0, 0, gain, 1, h_out, capture, H, eps, in, up, up_blocks, 1, M);
}

// grid: x = pair, y = 1024 elements of the row, then of the queries: every thread has all its loads in flight (one block per
// pair, an element per thread and pass, took 9.8 us; now 4.8).
__global__ __launch_bounds__(256) void put_aside_kernel(const int32_t* __restrict__ pairs, const float* __restrict__ x, float* __restrict__ x_out,
                                                       int H, const float* __restrict__ q, float* __restrict__ q_out, int D) {
  const size_t from = pairs[2 * blockIdx.x], to = pairs[2 * blockIdx.x + 1];
  const int nx = (H + 1023) / 1024, c = blockIdx.y < nx ? blockIdx.y : blockIdx.y - nx, n = (int)blockIdx.y < nx ? H : D;
  const float* in = (int)blockIdx.y < nx ? x + from * H : q + from * D;
  float* out = (int)blockIdx.y < nx ? x_out + to * H : q_out + to * D;
  float v[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = in[min(c * 1024 + e * 256 + (int)threadIdx.x, n - 1)];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const int i = c * 1024 + e * 256 + threadIdx.x;
    if (i < n) out[i] = v[e];
  }
}

void launch_put_aside(hipStream_t s, const int32_t* pairs, int n, const float* x, float* x_out, int H, const float* q, float* q_out, int D) {
  if (n > 0) put_aside_kernel<<<dim3(n, (H + 1023) / 1024 + (D + 1023) / 1024), 256, 0, s>>>(pairs, x, x_out, H, q, q_out, D);
}

__global__ __launch_bounds__(256) void repeat_rows_kernel(const float* __restrict__ in, float* __restrict__ out, int H, int group) {
  const size_t r = blockIdx.x;
  for (int i = threadIdx.x; i < H; i += 256) out[r * H + i] = in[r / group * H + i];
}

void launch_repeat_rows(hipStream_t s, const float* in, float* out, int M, int H, int group) {
  repeat_rows_kernel<<<M, 256, 0, s>>>(in, out, H, group);
}

// One wave per (row, head), four heads per block.  Lane i < d/2 owns the rotary pair (i, i + d/2).
template <bool BF16, int KVT>
__global__ __launch_bounds__(256) void qk_rope_append_kernel(const float* __restrict__ part, int S, size_t split_stride,
                                                            const void* __restrict__ q_gain,
                                                            const void* __restrict__ k_gain,
                                                            const float2* __restrict__ rope, const RowMeta* __restrict__ rows,
                                                            void* __restrict__ k_pool, void* __restrict__ v_pool,
                                                            float* __restrict__ q_out, int n_q, int n_kv, int d,
                                                            int qk_norm, float eps) {
  const int hh = blockIdx.x * 4 + (threadIdx.x >> 6), r = blockIdx.y, lane = threadIdx.x & 63;
  if (hh >= n_q + 2 * n_kv) return;  // wave-uniform; no barriers in this kernel
  const int half = d >> 1;
  const int n_tot = (n_q + 2 * n_kv) * d;
  const RowMeta rm = rows[r];
  const bool is_q = hh < n_q, is_k = !is_q && hh < n_q + n_kv;
  // Everything that depends only on the row's (seq, pos) is requested first, so that it travels together with the
  // partial sums instead of after them.
  const int64_t page = rm.page;
  const bool rotate = is_q || is_k;
  const float* head_part = part + (size_t)r * n_tot + (size_t)hh * d;
  const void* gain = qk_norm ? (is_q ? q_gain : k_gain) : nullptr;
  // lanes may own more than one pair when d/2 > 64 (without per-head normalisation only: the host rejects wider
  // normalised heads for this kernel)
  for (int i = lane; i < ((half + 63) & ~63); i += 64) {
    HeadPair hp = head_pair_load<BF16>(head_part, S, split_stride, d, i, rotate, rope + (size_t)rm.pos * half, gain);
    head_pair_finish(hp, d, rotate, qk_norm != 0, eps);
    if (i >= half) continue;
    if (is_q) {
      float* q = q_out + ((size_t)r * n_q + hh) * d;
      q[i] = hp.v0;
      q[i + half] = hp.v1;
    } else {
      const int hk = is_k ? hh - n_q : hh - n_q - n_kv;
      const int t = rm.pos & 15;
      kv_store<KVT>(is_k ? k_pool : v_pool, page, hk, n_kv, d, t, i, hp.v0, !is_k);
      kv_store<KVT>(is_k ? k_pool : v_pool, page, hk, n_kv, d, t, i + half, hp.v1, !is_k);
    }
  }
}

// The same for bf16 models, many rows and a finished projection (one partial): one block per row, its heads in groups of
// four per wave, so that a wave has the loads of four heads in flight and fetches the row's rotation and the gains once.
// Same arithmetic, same bits.  It moves 46 MB at 1024 rows: 19.7 -> 13.1 us.
template <int KVT>
__global__ __launch_bounds__(256) void qk_rope_append_rows_kernel(const float* __restrict__ part, const void* __restrict__ q_gain,
                                                                 const void* __restrict__ k_gain, const float2* __restrict__ rope, const RowMeta* __restrict__ rows,
                                                                 void* __restrict__ k_pool, void* __restrict__ v_pool,
                                                                 float* __restrict__ q_out, int n_q, int n_kv, int qk_norm, float eps) {
  constexpr int d = 128, half = 64;
  const int r = blockIdx.x, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int n_rot = n_q + n_kv, n_heads = n_rot + n_kv;
  const RowMeta rm = rows[r];
  const float* row_part = part + (size_t)r * n_heads * d;
  const float2 cs = rope[(size_t)rm.pos * half + lane];
  float gq[2] = {1.f, 1.f}, gk[2] = {1.f, 1.f};
  if (qk_norm) {
    gq[0] = bf2f(((const uint16_t*)q_gain)[lane]); gq[1] = bf2f(((const uint16_t*)q_gain)[lane + half]);
    gk[0] = bf2f(((const uint16_t*)k_gain)[lane]); gk[1] = bf2f(((const uint16_t*)k_gain)[lane + half]);
  }
  for (int h0 = 4 * wave; h0 < n_heads; h0 += 16) {
    float ld[4][2];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float* p = row_part + (size_t)min(h0 + u, n_heads - 1) * d;
      ld[u][0] = p[lane];
      ld[u][1] = p[lane + half];
    }
    HeadPair hp[4], raw[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      hp[u].v0 = 0.f + ld[u][0];  // the sum over one split
      hp[u].v1 = 0.f + ld[u][1];
      const bool is_q = h0 + u < n_q;
      hp[u].cs = cs;
      hp[u].g0 = is_q ? gq[0] : gk[0];
      hp[u].g1 = is_q ? gq[1] : gk[1];
      raw[u] = hp[u];
    }
    if (h0 < n_rot) head_pairs_finish<4>(hp, d, qk_norm != 0, eps);  // wave-uniform
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const int hh = h0 + u;
      if (hh >= n_heads) continue;
      if (hh < n_q) {
        float* q = q_out + ((size_t)r * n_q + hh) * d;
        q[lane] = hp[u].v0;
        q[lane + half] = hp[u].v1;
      } else {
        const bool is_k = hh < n_rot;
        const int hk = is_k ? hh - n_q : hh - n_rot, t = rm.pos & 15;
        kv_store<KVT>(is_k ? k_pool : v_pool, rm.page, hk, n_kv, d, t, lane, is_k ? hp[u].v0 : raw[u].v0, !is_k);
        kv_store<KVT>(is_k ? k_pool : v_pool, rm.page, hk, n_kv, d, t, lane + half, is_k ? hp[u].v1 : raw[u].v1, !is_k);
      }
    }
  }
}

void launch_qk_rope_append(hipStream_t s, const Geometry& g, const float* qkv_part, int S, const void* q_gain,
                           const void* k_gain, const float2* rope_table, const RowMeta* rows, void* k_pool_layer,
                           void* v_pool_layer, float* q_out, int M) {
  dim3 grid((g.n_q + 2 * g.n_kv + 3) / 4, M);
  size_t stride = (size_t)M * (g.n_q + 2 * g.n_kv) * g.head_dim;
  if (g.dtype == kBF16 && M >= 512 && S == 1) {  // fewer rows: one wave per head gives more waves (301 rows 8.2 us, by row 10.4)
    if (g.kv_fp8)
      qk_rope_append_rows_kernel<2><<<M, 256, 0, s>>>(qkv_part, q_gain, k_gain, rope_table, rows, k_pool_layer, v_pool_layer, q_out, g.n_q, g.n_kv, g.qk_norm, g.rms_eps);
    else
      qk_rope_append_rows_kernel<1><<<M, 256, 0, s>>>(qkv_part, q_gain, k_gain, rope_table, rows, k_pool_layer, v_pool_layer, q_out, g.n_q, g.n_kv, g.qk_norm, g.rms_eps);
    return;
  }
  if (g.dtype == kBF16 && g.kv_fp8)
    qk_rope_append_kernel<true, 2><<<grid, 256, 0, s>>>(qkv_part, S, stride, q_gain, k_gain, rope_table, rows,
                                                       k_pool_layer, v_pool_layer, q_out, g.n_q, g.n_kv,
                                                       g.head_dim, g.qk_norm, g.rms_eps);
  else if (g.dtype == kBF16)
    qk_rope_append_kernel<true, 1><<<grid, 256, 0, s>>>(qkv_part, S, stride, q_gain, k_gain, rope_table, rows,
                                                       k_pool_layer, v_pool_layer, q_out, g.n_q, g.n_kv,
                                                       g.head_dim, g.qk_norm, g.rms_eps);
  else
    qk_rope_append_kernel<false, 0><<<grid, 256, 0, s>>>(qkv_part, S, stride, q_gain, k_gain, rope_table, rows,
                                                        k_pool_layer, v_pool_layer, q_out, g.n_q, g.n_kv,
                                                        g.head_dim, g.qk_norm, g.rms_eps);
}

// ------------------------------------------------------------------------------------------------
// KV import: contiguous [n_tokens][n_kv][d] -> positions first_pos .. first_pos + n_tokens - 1 of one sequence.
// ------------------------------------------------------------------------------------------------
template <typename T, int KVT>
__global__ __launch_bounds__(256) void kv_import_kernel(const T* __restrict__ k_src, const T* __restrict__ v_src,
                                                        int first_pos, const int32_t* __restrict__ bt_row,
                                                        void* __restrict__ k_pool, void* __restrict__ v_pool, int n_kv,
                                                        int d) {
  const int tok = first_pos + blockIdx.x;  // position in the sequence; source token blockIdx.x
  const int64_t page = bt_row[tok >> 4];
  const int t = tok & 15;
  for (int i = threadIdx.x; i < n_kv * d; i += 256) {
    int hk = i / d, dd = i - hk * d;
    size_t src = (size_t)blockIdx.x * n_kv * d + i;
    kv_store<KVT>(k_pool, page, hk, n_kv, d, t, dd, load_as_float(k_src, src), false);
    kv_store<KVT>(v_pool, page, hk, n_kv, d, t, dd, load_as_float(v_src, src), true);
  }
}

void launch_kv_import(hipStream_t s, const Geometry& g, const void* k_src, const void* v_src, int first_pos, int n_tokens,
                      const int32_t* block_table_row, void* k_pool_layer, void* v_pool_layer) {
  if (n_tokens <= 0) return;
  if (g.dtype == kBF16 && g.kv_fp8)
    kv_import_kernel<uint16_t, 2><<<n_tokens, 256, 0, s>>>((const uint16_t*)k_src, (const uint16_t*)v_src, first_pos,
                                                           block_table_row, k_pool_layer, v_pool_layer, g.n_kv,
                                                           g.head_dim);
  else if (g.dtype == kBF16)
    kv_import_kernel<uint16_t, 1><<<n_tokens, 256, 0, s>>>((const uint16_t*)k_src, (const uint16_t*)v_src, first_pos,
                                                           block_table_row, k_pool_layer, v_pool_layer, g.n_kv,
                                                           g.head_dim);
  else
    kv_import_kernel<float, 0><<<n_tokens, 256, 0, s>>>((const float*)k_src, (const float*)v_src, first_pos,
                                                            block_table_row, k_pool_layer, v_pool_layer, g.n_kv,
                                                            g.head_dim);
}

// ------------------------------------------------------------------------------------------------
// Weight packing: row-major [N][K] bf16 -> fragment-major, each weight as its f16 image (the grid the matrix cores
// multiply on; see bf2_to_h2: exact from 2^-14 up, smaller magnitudes cut toward zero, same bytes per weight), so
// that no kernel spends an instruction on it.  One thread per 8 consecutive k.
// ------------------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void pack_weight_kernel(const uint4* __restrict__ src, uint4* __restrict__ dst, int N,
                                                          int K, int seg) {
  const size_t idx = (size_t)blockIdx.x * 256 + threadIdx.x;  // over N * K/8
  const int kg = K >> 3;
  if (idx >= (size_t)N * kg) return;
  const int n = (int)(idx / kg), k = (int)(idx - (size_t)n * kg) * 8;
  const uint4 w = src[idx];
  dst[weight_offset(n, k, K >> 6, seg) >> 3] = make_uint4(bf2_to_h2(w.x), bf2_to_h2(w.y), bf2_to_h2(w.z), bf2_to_h2(w.w));
}

void launch_pack_weight_bf16(hipStream_t s, const void* src, void* dst, int N, int K, int seg) {
  size_t total = (size_t)N * (K >> 3);
  pack_weight_kernel<<<(unsigned)((total + 255) / 256), 256, 0, s>>>((const uint4*)src, (uint4*)dst, N, K, seg);
}

}  // namespace rl

namespace rl {

// grid: x = layer (its copy of the partial page), then one more for the block-table row; y = fork.
constexpr int kForkThreads = 1024;
__global__ __launch_bounds__(kForkThreads) void fork_kernel(ForkBatch batch, int32_t* __restrict__ bt, int max_blocks, char* __restrict__ pool,
                                                   size_t layer_bytes, size_t page_bytes, int n_layers) {
  const ForkBatch::One f = batch.f[blockIdx.y];
  const int32_t* from = bt + (size_t)f.src * max_blocks;
  if ((int)blockIdx.x == n_layers) {
    int32_t* to = bt + (size_t)f.dst * max_blocks;
    for (int b = threadIdx.x; b < f.full; b += kForkThreads) to[b] = from[b];
    if (threadIdx.x == 0 && f.page >= 0) to[f.full] = f.page;
    return;
  }
  if (f.page < 0) return;
  char* base = pool + (size_t)blockIdx.x * layer_bytes;
  const uint4* s = (const uint4*)(base + (size_t)from[f.full] * page_bytes);
  uint4* d = (uint4*)(base + (size_t)f.page * page_bytes);
#pragma unroll 4
  for (size_t i = threadIdx.x; i < page_bytes / 16; i += kForkThreads) d[i] = s[i];
}

void launch_fork(hipStream_t s, const ForkBatch& batch, int32_t* block_table, int max_blocks, void* kv_pool, size_t layer_bytes,
                 size_t page_bytes, int n_layers) {
  fork_kernel<<<dim3(n_layers + 1, batch.n), kForkThreads, 0, s>>>(batch, block_table, max_blocks, (char*)kv_pool, layer_bytes, page_bytes, n_layers);
}

}  // namespace rl

namespace rl {

__global__ void scatter_f32_kernel(const float* __restrict__ src, const int32_t* __restrict__ idx, float* __restrict__ out, int n) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i < n && idx[i] >= 0) out[idx[i]] = src[i];
}

void launch_scatter_f32(hipStream_t s, const float* src, const int32_t* idx, float* out, int n) {
  if (n <= 0) return;
  scatter_f32_kernel<<<(n + 255) / 256, 256, 0, s>>>(src, idx, out, n);
}

}  // namespace rl
