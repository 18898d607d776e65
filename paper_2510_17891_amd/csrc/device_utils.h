// Small device helpers shared by the gfx950 kernels: bf16 packing, wave64 reductions, vector types.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rl {

typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef float f32x16_t __attribute__((ext_vector_type(16)));

constexpr int kWave = 64;
constexpr int kPageTokens = 16;  // tokens per KV page

// fp32 -> bf16 bits, round to nearest even (finite inputs).
__device__ __forceinline__ uint32_t f2bf(float x) {
  uint32_t u = __float_as_uint(x);
  u += 0x7fffu + ((u >> 16) & 1u);
  return u >> 16;
}
__device__ __forceinline__ float bf2f(uint32_t b) { return __uint_as_float(b << 16); }
__device__ __forceinline__ uint32_t pack2bf(float lo, float hi) { return f2bf(lo) | (f2bf(hi) << 16); }

// The projections multiply on the f16 grid: the packed weights hold the f16 image of the model's bf16 weights (made
// once, when they are packed), activations are written as f16 by their producers.  f16 keeps 11 significant bits against bf16's 8, so the rounding of an
// activation entering a projection is 8 times smaller, at the same bytes and the same matrix-core rate.
//
// Two bf16 (one 32-bit word) -> two f16.  Exact for 2^-14 <= |w| <= 65504 (a bf16 significand fits an f16 one);
// smaller magnitudes are cut toward zero on the f16 subnormal grid (absolute error < 2^-24), larger ones end at
// +-65504.
__device__ __forceinline__ uint32_t bf2_to_h2(uint32_t w) {
  const float lo = __uint_as_float(w << 16), hi = __uint_as_float(w & 0xffff0000u);
  return __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_pkrtz(lo, hi));
}
// fp32 -> f16 bits, round to nearest even, finite values beyond the f16 range end at +-65504 (NaN stays NaN).
__device__ __forceinline__ uint32_t f2h(float x) {
  x = x > 65504.0f ? 65504.0f : (x < -65504.0f ? -65504.0f : x);
  return (uint32_t)__builtin_bit_cast(uint16_t, (_Float16)x);
}
__device__ __forceinline__ uint32_t pack2h(float lo, float hi) { return f2h(lo) | (f2h(hi) << 16); }

// Storage-type accessors used by the dtype-generic kernels.
__device__ __forceinline__ float load_as_float(const float* p, size_t i) { return p[i]; }
__device__ __forceinline__ float load_as_float(const uint16_t* p, size_t i) { return bf2f(p[i]); }
__device__ __forceinline__ void store_from_float(float* p, size_t i, float v) { p[i] = v; }
__device__ __forceinline__ void store_from_float(uint16_t* p, size_t i, float v) { p[i] = (uint16_t)f2bf(v); }

// Values of the lanes `mask` apart (a power of two, a constant once loops are unrolled; all 64 lanes active).  Within 16 lanes
// these are data-parallel-primitive moves, beyond them gfx950's swaps of 16- and 32-lane halves: a few cycles, where an
// exchange through the LDS crossbar (__shfl_xor) takes over a hundred, and a reduction chains six of them.
struct LanePair {
  uint32_t a, b;  // own and other value, in an order that is the same in both lanes for masks 16 and 32
};
__device__ __forceinline__ LanePair lane_pair_bits(uint32_t v, int mask) {
  const int x = (int)v;
  switch (mask) {
    case 1: return {v, (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0xB1, 0xf, 0xf, true)};  // quad_perm 1 0 3 2
    case 2: return {v, (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x4E, 0xf, 0xf, true)};  // quad_perm 2 3 0 1
    case 4: {  // row_half_mirror (lane ^ 7), then quad_perm 3 2 1 0 (lane ^ 3)
      const int h = __builtin_amdgcn_update_dpp(0, x, 0x141, 0xf, 0xf, true);
      return {v, (uint32_t)__builtin_amdgcn_update_dpp(0, h, 0x1B, 0xf, 0xf, true)};
    }
    case 8: return {v, (uint32_t)__builtin_amdgcn_update_dpp(0, x, 0x128, 0xf, 0xf, true)};  // row_ror 8
    case 16: {
      const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
      return {r[0], r[1]};
    }
    default: {
      const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
      return {r[0], r[1]};
    }
  }
}
__device__ __forceinline__ uint32_t lane_xor(uint32_t v, int mask) {
  const LanePair p = lane_pair_bits(v, mask);
  return mask >= 16 && (threadIdx.x & mask) ? p.a : p.b;
}
__device__ __forceinline__ int lane_xor(int v, int mask) { return (int)lane_xor((uint32_t)v, mask); }
__device__ __forceinline__ float lane_xor(float v, int mask) { return __uint_as_float(lane_xor(__float_as_uint(v), mask)); }
__device__ __forceinline__ unsigned long long lane_xor(unsigned long long v, int mask) {
  return ((unsigned long long)lane_xor((uint32_t)(v >> 32), mask) << 32) | lane_xor((uint32_t)v, mask);
}
// v of this lane and the one `mask` apart: sum and maximum.
__device__ __forceinline__ float lane_add(float v, int mask) {
  const LanePair p = lane_pair_bits(__float_as_uint(v), mask);
  return __uint_as_float(p.a) + __uint_as_float(p.b);
}
__device__ __forceinline__ float lane_max(float v, int mask) {
  const LanePair p = lane_pair_bits(__float_as_uint(v), mask);
  return fmaxf(__uint_as_float(p.a), __uint_as_float(p.b));
}

// fn(kFirst), fn(kFirst / 2), ..., fn(1): the steps of a reduction, each with its mask as a constant.
template <int kFirst = 32, typename F>
__device__ __forceinline__ void each_mask(F fn) {
  fn(kFirst);
  if constexpr (kFirst > 1) each_mask<kFirst / 2>(fn);
}

__device__ __forceinline__ float wave_sum(float v) {
  each_mask([&](int o) __attribute__((always_inline)) { v = lane_add(v, o); });
  return v;
}
__device__ __forceinline__ float wave_max(float v) {
  each_mask([&](int o) __attribute__((always_inline)) { v = lane_max(v, o); });
  return v;
}

}  // namespace rl
