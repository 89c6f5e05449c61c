// Device code shared by the kernels of libmoe_gfx950: vector types, activations, LDS reads, the wait on a flag.
#pragma once
#include "moe_internal.h"

namespace moe {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) short s16x4;
typedef __attribute__((ext_vector_type(8))) short s16x8;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;
typedef __attribute__((ext_vector_type(2))) uint32_t u32x2;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;

enum { MODE_L0_GELU = 0, MODE_L0_SWIGLU = 1, MODE_L1 = 2 };

// Two transposing reads: lane gets B[k0..k0+3][n] and B[k0+4..k0+7][n] of its column n.
__device__ __forceinline__ bf16x8 lds_read_b(uint32_t a0, uint32_t a1) {
  s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(uintptr_t)a0);
  s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(uintptr_t)a1);
  s16x8 v = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
  return __builtin_bit_cast(bf16x8, v);
}

// Tells the compiler that a pointer / integer is the same in every lane (keeps it in scalar registers).
__device__ __forceinline__ const char* uniform(const char* ptr) {
  const uint64_t v = (uint64_t)(uintptr_t)ptr;
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return (const char*)(uintptr_t)(((uint64_t)hi << 32) | lo);
}
__device__ __forceinline__ int uniform(int v) { return __builtin_amdgcn_readfirstlane(v); }

// GELU in its erf form, 0.5 v (1 + erf(v / sqrt 2)).  erf is evaluated with the 5-term formula 7.1.26 of Abramowitz and
// Stegun's Handbook of Mathematical Functions, the rational
// approximation 1 - (a1 t + ... + a5 t^5) exp(-z^2), t = 1 / (1 + 0.3275911 z) (absolute error below 1.5e-7,
// far under the bf16 rounding of the result); it needs a handful of registers, which matters next to 256
// live accumulators.
__device__ __forceinline__ float gelu_erf(float v) {
  const float z = fabsf(v) * 0.70710678118654752f;
  const float t = __builtin_amdgcn_rcpf(1.0f + 0.3275911f * z);
  float poly = 1.061405429f;
  poly = poly * t - 1.453152027f;
  poly = poly * t + 1.421413741f;
  poly = poly * t - 0.284496736f;
  poly = poly * t + 0.254829592f;
  const float erf_abs = 1.0f - poly * t * __builtin_amdgcn_exp2f(z * z * -1.4426950408889634f);
  const float erf_v = v < 0.f ? -erf_abs : erf_abs;
  return 0.5f * v * (1.0f + erf_v);
}
// v * sigmoid(v) with the hardware exp2 and reciprocal (about 1 ulp each; the result is rounded to bf16 anyway).
__device__ __forceinline__ float silu(float v) {
  return v * __builtin_amdgcn_rcpf(1.0f + __builtin_amdgcn_exp2f(v * -1.4426950408889634f));
}

// ---------------------------------------------------------------------------------------------
// Tiling of an expert's rows: as many tiles of tile_m rows as fit, then one tile for the remainder.  A tile's height class is the
// lowest of 64, 128 and 256 rows that holds it.  (A remainder of
// 129 to 192 rows, for which there is a variant, is not split into a 128- and a 64-row tile: every tile of a column streams
// the expert's weights, which costs what the matrix cores need for about 240 rows.  160 rows for each of 16
// experts with F = 6400: 941 -> 611 us, 400 rows 1385 -> 1022.)
// ---------------------------------------------------------------------------------------------
__device__ inline int height_class(int rows) { return rows <= 64 ? 0 : (rows <= 128 ? 1 : 2); }
// Rows of the kernel variant that computes a tile.
__device__ inline int variant_rows(int rows) { return rows <= 64 ? 64 : (rows <= 128 ? 128 : (rows <= 192 ? 192 : 256)); }

// Waves of the layer0 schedule (order 2) of this forward, decided by one wavefront for everybody: the plan's number, or
// one -- the order of resident input -- when every source segment has arrived by now (waves cost the weight reuse: layer0
// of 16384 tokens of 16 experts with F = 6400 takes 3050 us against 2605, of 2047 tokens of 8 with F = 3584 284 against
// 254).  A flag raised later than this only costs that.
__device__ inline int waves_now(const IndexParams& p, int lane) {
  if (p.seg_ready == nullptr) return p.layer0_waves;
  bool missing = false;
  if (lane < p.s.S && p.seg_offsets[lane + 1] > p.seg_offsets[lane])
    missing = __hip_atomic_load(&p.seg_ready[lane], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) < p.ready_epoch;
  return __ballot(missing) != 0 ? p.layer0_waves : 1;
}

// Wait until *flag >= want.  Returns false if the spin limit (when set) ran out.
__device__ __forceinline__ bool spin_until_ge(const uint32_t* flag, uint32_t want, uint32_t spin_limit) {
  uint32_t polls = 0;
  while (__hip_atomic_load(flag, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM) < want) {
    __builtin_amdgcn_s_sleep(8);
    if (spin_limit && ++polls >= spin_limit) return false;
  }
  return true;
}

}  // namespace moe
