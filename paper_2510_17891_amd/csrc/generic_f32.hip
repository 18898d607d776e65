// fp32 kernels for models stored in fp32 (hidden and ffn multiples of 8, any even head_dim up to 128 with any number of
// heads): projections on the vector ALUs and paged attention.  These serve the small full-precision configuration, where every tensor fits in cache and a step is a
// chain of launches that each last about as long as a few dependent memory round trips.  They are therefore written for
// few launches (norm and residual inside the projections, rotation and KV append inside the attention) and for having
// all loads of a launch in flight at once.  A decode step of 4 rows through two layers of 256 hidden dimensions, sampling
// included: 48 us in 13 launches (150 us in 23 with separate norms, rotation and append, projections with one 4-byte load
// per lane and a single wave per attention head; 57 us with weights that waited pass by pass, an attention that asked for
// keys and values behind the query, and two launches of the sampler).
#include <type_traits>

#include "device_utils.h"
#include "kernels.h"
#include "rope_device.h"

namespace rl {

namespace {

// Sums of R values over the 64 lanes, the total of value i in lanes i, i + R, ...: every exchange step halves the values a
// lane still carries (7 exchanges for 4 values instead of 24).  Each value is added up in the same tree whatever R is.
template <int R>
__device__ __forceinline__ float wave_sums(const float (&v)[R], int lane) {
  float a[R];
#pragma unroll
  for (int i = 0; i < R; ++i) a[i] = v[i];
  int n = R;
#pragma unroll
  for (int mask = 1; mask < 64; mask <<= 1) {
    if (n > 1) {
      const bool up = (lane & mask) != 0;
#pragma unroll
      for (int i = 0; i < R / 2; ++i)
        if (i < n / 2) {
          const float keep = up ? a[2 * i + 1] : a[2 * i], send = up ? a[2 * i] : a[2 * i + 1];
          a[i] = keep + lane_xor(send, mask);
        }
      n >>= 1;
    } else {
      a[0] = lane_add(a[0], mask);
    }
  }
  return a[0];
}

// One wave per C output columns from C n on (4 waves per block) and R rows: lane l takes VEC elements from VEC l on of
// every 64 VEC.  K % VEC == 0.  VEC is 4 except for the O projection of an odd number of heads whose head_dim is no
// multiple of four: there K is only even, rows begin on 8-byte boundaries, and a group of four would reach into the next row.
// kEpiSwiGLU: W has 2N rows (gate then up); out[m][n] = silu(gate)*up.  kEpiResidual: out[m][n] += product.
// gain (may be null, not used with kEpiResidual): the rows are RMS-normalised first, x * rsqrt(mean(x^2) + eps) * gain; every wave forms the row's
// mean square from the elements it holds anyway.  A row's result depends neither on R and C nor on the rows beside it.
template <int EPI, int R, int C, int VEC>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ X, const float* __restrict__ W,
                                                       float* __restrict__ out, int M, int N, int K, int m_tiles,
                                                       const float* __restrict__ gain, float eps) {
  typedef float vec_t __attribute__((ext_vector_type(VEC)));
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  // Consecutive blocks go to the eight dies in turn: the row tiles of one column tile follow each other on one die, whose
  // L2 then gives the weights to all but the first of them.
  const int j = blockIdx.x >> 3;
  const int m0 = j % m_tiles * R, n = (((j / m_tiles) * 8 + (blockIdx.x & 7)) * 4 + wave) * C;
  if (n >= N) return;
  const float* w0[C];
  const float* w1[C];  // only read for SwiGLU
#pragma unroll
  for (int c = 0; c < C; ++c) {
    w0[c] = W + (size_t)min(n + c, N - 1) * K;
    w1[c] = w0[c] + (size_t)N * K;
  }
  float a0[C][R], a1[C][R], ss[R], old[C];
#pragma unroll
  for (int c = 0; c < C; ++c)  // what the product is added to, requested ahead of it
    old[c] = EPI == kEpiResidual ? out[(size_t)min(m0 + min(lane, R - 1), M - 1) * N + min(n + c, N - 1)] : 0.f;
#pragma unroll
  for (int i = 0; i < R; ++i) {
    ss[i] = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c) a0[c][i] = a1[c][i] = 0.f;
  }
  // One pass: 64 VEC elements of the weights and of the rows, requested together and used together, up to kFlight passes at
  // a time (a pass that waits for the one before costs a round trip to memory).  Elements past the end are read from
  // the row's start and count as zero.
  struct Pass { vec_t u[C], v[C], g, x[R]; };
  constexpr bool kNorm = EPI != kEpiResidual;  // what is added to the residual stream has no norm in front
  const float* const gains = gain ? gain : w0[0];  // read and not used without a norm
  auto load = [&](Pass& p, int k, bool all) __attribute__((always_inline)) {
    const bool in = all || k < K;
    const int kk = in ? k : 0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
      p.u[c] = *(const vec_t*)(w0[c] + kk);
      p.v[c] = 0.f;
      if (EPI == kEpiSwiGLU) p.v[c] = *(const vec_t*)(w1[c] + kk);
    }
    if (kNorm) p.g = *(const vec_t*)(gains + kk);
#pragma unroll
    for (int i = 0; i < R; ++i) p.x[i] = *(const vec_t*)(X + (size_t)min(m0 + i, M - 1) * K + kk);
  };
  auto use = [&](Pass& p, int k, bool all) __attribute__((always_inline)) {
    if (!all && k >= K) {
#pragma unroll
      for (int c = 0; c < C; ++c) p.u[c] = p.v[c] = 0.f;
#pragma unroll
      for (int i = 0; i < R; ++i) p.x[i] = 0.f;
      if (kNorm) p.g = 0.f;
    }
    vec_t g = 1.f;
    if (kNorm) g = p.g;
    const auto& u = p.u;
    const auto& v = p.v;
#pragma unroll
    for (int i = 0; i < R; ++i) {
      vec_t x = p.x[i];
      if (kNorm && gain) {
#pragma unroll
        for (int e = VEC - 1; e >= 0; --e) ss[i] = fmaf(x[e], x[e], ss[i]);
        x *= g;
      }
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = VEC - 1; e >= 0; --e) {
          a0[c][i] = fmaf(u[c][e], x[e], a0[c][i]);
          if (EPI == kEpiSwiGLU) a1[c][i] = fmaf(v[c][e], x[e], a1[c][i]);
        }
    }
  };
  // Four passes of eight rows leave two waves on a SIMD: 8 rows through 2048 x 5504 and 2048 x 2048 20.1 us, with two passes 15.7.
  constexpr int kFlight = C == 1 && R < 8 ? 4 : 2, kPass = 64 * VEC;
  int k = VEC * lane, left = (K + kPass - 1) / kPass;
  auto passes = [&](auto nc) __attribute__((always_inline)) {
    constexpr int n = decltype(nc)::value;
    Pass p[n];
#pragma unroll
    for (int e = 0; e < n; ++e) load(p[e], k + e * kPass, e + 1 < n);
#pragma unroll
    for (int e = 0; e < n; ++e) use(p[e], k + e * kPass, e + 1 < n);
    k += n * kPass;
    left -= n;
  };
  while (left >= kFlight) passes(std::integral_constant<int, kFlight>{});
  if constexpr (kFlight > 2) {
    if (left == 3) passes(std::integral_constant<int, 3>{});
    else if (left == 2) passes(std::integral_constant<int, 2>{});
  }
  if (left == 1) passes(std::integral_constant<int, 1>{});
  float inv = 1.f;
  if (kNorm && gain) inv = 1.0f / sqrtf(wave_sums<R>(ss, lane) / (float)K + eps);
#pragma unroll
  for (int c = 0; c < C; ++c) {
    float s0 = wave_sums<R>(a0[c], lane), s1 = 0.f;
    if (EPI == kEpiSwiGLU) s1 = wave_sums<R>(a1[c], lane);
    if (gain) {
      s0 *= inv;
      s1 *= inv;
    }
    const int m = m0 + lane;
    if (lane >= R || m >= M || n + c >= N) continue;
    float* o = out + (size_t)m * N + n + c;
    if (EPI == kEpiSwiGLU) *o = s0 / (1.0f + expf(-s0)) * s1;
    else if (EPI == kEpiResidual) *o = old[c] + s0;
    else *o = s0;
  }
}

struct F32Append {
  const float* qkv;  // [M][(n_q + 2 n_kv) * d]
  const float* q_gain;
  const float* k_gain;
  const float2* rope;
  float eps;
};

// One block of four waves per (row, q head), keys in tiles of 256: one key per thread for the scores; for the weighted
// sum a thread owns VEC dims and every (256 / (d / VEC))-th key; online softmax across tiles.  d <= 128, d % VEC == 0.
// APPEND (one row per sequence): the block forms its query and the row's new key and value from the QKV projection, uses
// the latter two from LDS, and the first head of the group writes them to the row's page.
// What bounds it is the chain of round trips in small batches and the keys' way through the caches in large ones.  So the
// pages are looked up and a thread's first kFirst values requested before the scores (for the first tile the pages, and the
// values, before the query is formed); a key comes in pieces of ND loads in flight, which leaves the registers for three and
// more blocks per compute unit; and everything that may be in a page is loaded from there, the new key and value replacing
// it in registers, because a pointer that may lead to LDS as well as to memory makes every load wait for both.  Kernel
// times (us) with such pointers -> with whole keys of up to 128 dims requested ahead of the query -> now: 4 rows of 70 keys of
// 64 dims 7.6 -> 7.0 -> 6.8, of 250 12.1 -> 11.8 -> 9.6, of 1500 57.9 -> 47.8 -> 37.0; 4 rows of 250 keys of 128 dims 17.8 -> 19.0 -> 14.1,
// of 126 dims 22.9 -> 28.1 -> 15.0; 64 rows of 600 keys of 64 dims 66 -> 69 -> 59, of 128 117 -> 131 -> 106, of 62 59 -> 53 -> 36.
// Finished rows (scoring, prefill), whose values are not requested ahead: 64 rows of 600 keys of 128 dims 31 -> 50 -> 30, of 64 18 -> 22 -> 18.
template <bool APPEND, int VEC, int ND>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float* __restrict__ q, const RowMeta* __restrict__ rows,
                                                       const int32_t* __restrict__ block_table, int max_blocks,
                                                       float* k_pool, float* v_pool, float* __restrict__ o_out, int n_q,
                                                       int n_kv, int d, float scale, F32Append ap) {
  typedef float vec_t __attribute__((ext_vector_type(VEC)));
  constexpr int kFirst = 4;
  __shared__ __align__(16) float qs[128], kn[128], vn[128], ps[256], part[256 * VEC];
  __shared__ float red[8];
  const int h = blockIdx.x, r = blockIdx.y, tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const RowMeta rm = rows[r];
  const int ctx = rm.pos + 1, group = n_q / n_kv, hk = h / group;
  const int32_t* bt = block_table + (size_t)rm.seq * max_blocks;
  const size_t page_elems = (size_t)kPageTokens * d;
  const int nd = d / VEC, groups = 256 / nd, dim = (tid % nd) * VEC, grp = tid / nd;
  const auto row_of = [&](const float* pool, int key, int page) __attribute__((always_inline)) {
    return pool + ((size_t)page * n_kv + hk) * 2 * page_elems + (size_t)(key & 15) * d;
  };
  vec_t acc = 0.f;
  float m_run = -INFINITY, l_run = 0.f;
  for (int kb = 0; kb < ctx; kb += 256) {
    const int key = min(kb + tid, ctx - 1);  // keys beyond the context repeat the last one and have no weight
    const float* const kp = row_of(k_pool, key, bt[key >> 4]);
    const bool has_keys = kb + 64 * wave < ctx;  // wave-uniform
    int v_key[kFirst], v_page[kFirst];
    if constexpr (APPEND) {
#pragma unroll
      for (int i = 0; i < kFirst; ++i) {
        v_key[i] = min(kb + grp + i * groups, ctx - 1);
        v_page[i] = bt[v_key[i] >> 4];
      }
    }
    HeadPair hp;
    const bool forms = APPEND && kb == 0 && wave < 3;  // query, new key, new value: one wave each
    const bool norm = ap.q_gain != nullptr && wave < 2;
    const int half = d >> 1;
    if (forms) {
      const int head = wave == 0 ? h : wave == 1 ? n_q + hk : n_q + n_kv + hk;
      hp = head_pair_load<false>(ap.qkv + ((size_t)r * (n_q + 2 * n_kv) + head) * d, 1, 0, d, lane, wave < 2,
                                 ap.rope + (size_t)rm.pos * half, norm ? (wave == 0 ? ap.q_gain : ap.k_gain) : nullptr);
    }
    vec_t vr[kFirst];
    if constexpr (APPEND) {
#pragma unroll
      for (int i = 0; i < kFirst; ++i)
        if (kb + i * groups < ctx) vr[i] = *(const vec_t*)(row_of(v_pool, v_key[i], v_page[i]) + dim);
    }
    if (kb == 0) {
      if (forms) {
        head_pair_finish(hp, d, wave < 2, norm, ap.eps);
        if (lane < half) {
          float* s = wave == 0 ? qs : wave == 1 ? kn : vn;
          s[lane] = hp.v0;
          s[lane + half] = hp.v1;
          if (wave > 0 && h == hk * group) {
            float* p = (wave == 1 ? k_pool : v_pool) + ((size_t)rm.page * n_kv + hk) * 2 * page_elems + (size_t)(rm.pos & 15) * d;
            p[lane] = hp.v0;
            p[lane + half] = hp.v1;
          }
        }
      }
      if (!APPEND)
        for (int i = tid; i < d; i += 256) qs[i] = q[((size_t)r * n_q + h) * d + i];
      __syncthreads();
    }
    vec_t dot = 0.f;
    if constexpr (!APPEND) {
      if (kb + tid < ctx) {
#pragma unroll 8
        for (int i = 0; i < d; i += VEC) dot += *(const vec_t*)(qs + i) * *(const vec_t*)(kp + i);
      }
    } else if (has_keys) {
      vec_t kr[ND];
      const auto load = [&](int first, int last) __attribute__((always_inline)) {  // pieces beyond `last` repeat it
#pragma unroll
        for (int i = 0; i < ND; ++i) kr[i] = *(const vec_t*)(kp + min(first + i, last) * VEC);
        if (key == rm.pos) {  // the new key is not in its page yet
#pragma unroll
          for (int i = 0; i < ND; ++i) kr[i] = *(const vec_t*)(kn + min(first + i, last) * VEC);
        }
      };
      int first = 0;
      for (; first + ND <= nd; first += ND) {
        load(first, first + ND - 1);
#pragma unroll
        for (int i = 0; i < ND; ++i) dot += *(const vec_t*)(qs + (first + i) * VEC) * kr[i];
      }
      if (first < nd) {
        load(first, nd - 1);
#pragma unroll
        for (int i = 0; i < ND; ++i)
          if (first + i < nd) dot += *(const vec_t*)(qs + (first + i) * VEC) * kr[i];
      }
    }
    float sc = dot[0];
#pragma unroll
    for (int e = 1; e < VEC; ++e) sc += dot[e];
    sc = kb + tid < ctx ? sc * scale : -INFINITY;
    float mx = wave_max(sc);
    if (lane == 0) red[wave] = mx;
    __syncthreads();
    const float m_new = fmaxf(m_run, fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3])));
    const float p = expf(sc - m_new);
    ps[tid] = p;
    const float sum = wave_sum(p);
    if (lane == 0) red[4 + wave] = sum;
    __syncthreads();
    const float alpha = expf(m_run - m_new);
    l_run = l_run * alpha + ((red[4] + red[5]) + (red[6] + red[7]));
    m_run = m_new;
    acc *= alpha;
    if (grp < groups) {
      const int nk = min(256, ctx - kb);
      if constexpr (APPEND) {
#pragma unroll
        for (int i = 0; i < kFirst; ++i) {
          const int t = grp + i * groups;
          if (t < nk) acc += ps[t] * (kb + t == rm.pos ? *(const vec_t*)(vn + dim) : vr[i]);
        }
      }
#pragma unroll 4
      for (int t = grp + (APPEND ? kFirst * groups : 0); t < nk; t += groups) {
        const int kt = kb + t;
        vec_t v = *(const vec_t*)(row_of(v_pool, kt, bt[kt >> 4]) + dim);
        if (APPEND && kt == rm.pos) v = *(const vec_t*)(vn + dim);
        acc += ps[t] * v;
      }
    }
    __syncthreads();
  }
  if (grp < groups) *(vec_t*)(part + grp * d + dim) = acc;  // groups * d <= 256 * VEC
  __syncthreads();
  const float inv = 1.0f / l_run;
  for (int i = tid; i < d; i += 256) {
    float s = 0.f;
    for (int g = 0; g < groups; ++g) s += part[g * d + i];
    o_out[((size_t)r * n_q + h) * d + i] = s * inv;
  }
}

template <int R, int C, int VEC>
void launch_gemm_rows(hipStream_t s, const float* X, const float* W, float* out, int M, int N, int K, int epi, const float* gain,
                      float eps) {
  const int m_tiles = (M + R - 1) / R, n_tiles = (N + 4 * C - 1) / (4 * C);
  const dim3 grid((n_tiles + 7) / 8 * 8 * m_tiles);
  if (epi == kEpiSwiGLU)
    gemm_f32_kernel<kEpiSwiGLU, R, C, VEC><<<grid, 256, 0, s>>>(X, W, out, M, N, K, m_tiles, gain, eps);
  else if (epi == kEpiResidual)
    gemm_f32_kernel<kEpiResidual, R, C, VEC><<<grid, 256, 0, s>>>(X, W, out, M, N, K, m_tiles, gain, eps);
  else
    gemm_f32_kernel<kEpiPartial, R, C, VEC><<<grid, 256, 0, s>>>(X, W, out, M, N, K, m_tiles, gain, eps);
}

template <int VEC>
void launch_gemm_vec(hipStream_t s, const float* X, const float* W, float* out, int M, int N, int K, int epi, const float* gain,
                     float eps) {
  // rows per wave: the smallest of 1, 4 and 8 that holds the batch (rows beyond it would be computed for nothing), 8 beyond,
  // where a wave also takes two columns: the rows then come from L1 once for both, and so does the mean square.  With two
  // layers of 2048 hidden dimensions a decode step of 64 rows takes 1.26 ms (3.15 with one column, 3.48 with the row tiles
  // one after the other as well) and a prefill of 900 tokens 9.9 ms (22.1, 26.0); of 256 dimensions 0.09 and 0.64 ms
  // (0.13, 0.93).  Four columns: 1.00, 8.4, 0.10, 0.65.
  if (M == 1) launch_gemm_rows<1, 1, VEC>(s, X, W, out, M, N, K, epi, gain, eps);
  else if (M <= 4) launch_gemm_rows<4, 1, VEC>(s, X, W, out, M, N, K, epi, gain, eps);
  else if (M <= 8) launch_gemm_rows<8, 1, VEC>(s, X, W, out, M, N, K, epi, gain, eps);
  else launch_gemm_rows<8, 2, VEC>(s, X, W, out, M, N, K, epi, gain, eps);
}

}  // namespace

void launch_gemm_f32(hipStream_t s, const float* X, const float* W, float* out, int M, int N, int K, int epi, const float* gain,
                     float eps) {
  if (K % 4 == 0) launch_gemm_vec<4>(s, X, W, out, M, N, K, epi, gain, eps);
  else launch_gemm_vec<2>(s, X, W, out, M, N, K, epi, gain, eps);
}

void launch_attn_f32(hipStream_t s, const Geometry& g, const float* q, const RowMeta* rows, const int32_t* block_table,
                     void* k_pool_layer, void* v_pool_layer, float* o_out, int M, const AttnAppend* append) {
  const dim3 grid(g.n_q, M);
  F32Append ap = {};
  if (append) ap = F32Append{append->qkv_part, (const float*)append->q_gain, (const float*)append->k_gain, append->rope_table, g.rms_eps};
  const float scale = 1.0f / sqrtf((float)g.head_dim);
#define RL_ATTN_F32(VEC, ND)                                                                                         \
  do {                                                                                                               \
    if (append)                                                                                                      \
      attn_f32_kernel<true, VEC, ND><<<grid, 256, 0, s>>>(q, rows, block_table, g.max_blocks, (float*)k_pool_layer,  \
                                                          (float*)v_pool_layer, o_out, g.n_q, g.n_kv, g.head_dim, scale, ap); \
    else                                                                                                             \
      attn_f32_kernel<false, VEC, ND><<<grid, 256, 0, s>>>(q, rows, block_table, g.max_blocks, (float*)k_pool_layer, \
                                                           (float*)v_pool_layer, o_out, g.n_q, g.n_kv, g.head_dim, scale, ap); \
  } while (0)
  if (g.head_dim % 4 == 0 && g.head_dim <= 16) RL_ATTN_F32(4, 4);
  else if (g.head_dim % 4 == 0) RL_ATTN_F32(4, 8);  // with sixteen loads in flight heads of 96 and 128 dims lose up to a fifth
  else RL_ATTN_F32(2, 16);  // an even head_dim: pairs keep the loads aligned
#undef RL_ATTN_F32
}

}  // namespace rl
