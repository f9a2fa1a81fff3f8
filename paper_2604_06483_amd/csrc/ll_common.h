// Shared device/host helpers of the HIP library (gfx950 only).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "ll.h"

namespace ll {

// Records a failed HIP call for ll_last_hip_error() and returns LL_EHIP.
int hip_failed(hipError_t e);

#define LL_HIP_CHECK(expr)                         \
  do {                                             \
    hipError_t e__ = (expr);                       \
    if (e__ != hipSuccess) return ll::hip_failed(e__); \
  } while (0)

inline size_t align_up(size_t x, size_t a) { return (x + a - 1) / a * a; }

constexpr int kWave = 64;

// ---- bf16 <-> fp32 on the device ------------------------------------------------------
// A bf16 value is the upper half of an fp32 word, so widening is a shift.
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef float f32x2_t __attribute__((ext_vector_type(2)));

// Two fp32 -> packed bf16 pair, round-to-nearest-even (one v_cvt_pk_bf16_f32 on gfx950).
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
  f32x2_t f = {lo, hi};
  bf16x2_t b = __builtin_convertvector(f, bf16x2_t);
  return __builtin_bit_cast(uint32_t, b);
}

// The value of lane l ^ OFF, combined with the lane's own by f (commutative), without a trip through LDS: six steps of an
// LDS exchange are some 600 cycles of waiting, six of these 60.  All lanes of the wavefront have to be on.
template <int CTRL>
__device__ __forceinline__ uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_mov_dpp((int)x, CTRL, 0xF, 0xF, true);
}
template <int OFF, class F>
__device__ __forceinline__ uint32_t with_lane_xor(uint32_t x, F f) {
  static_assert(OFF == 1 || OFF == 2 || OFF == 4 || OFF == 8 || OFF == 16 || OFF == 32, "one bit of the lane number");
  if constexpr (OFF == 32) {
    const auto p = __builtin_amdgcn_permlane32_swap(x, x, false, false);
    return f(p[0], p[1]);
  } else if constexpr (OFF == 16) {
    const auto p = __builtin_amdgcn_permlane16_swap(x, x, false, false);
    return f(p[0], p[1]);
  } else if constexpr (OFF == 8) {
    return f(x, dpp<0x128>(x));             // row_ror:8
  } else if constexpr (OFF == 4) {
    return f(x, dpp<0x1B>(dpp<0x141>(x)));  // row_half_mirror, then each quad reversed: l ^ 7 ^ 3
  } else {
    return f(x, dpp<OFF == 2 ? 0x4E : 0xB1>(x));
  }
}
template <class F>
__device__ __forceinline__ uint32_t wave_combine(uint32_t x, F f) {
  x = with_lane_xor<32>(x, f);
  x = with_lane_xor<16>(x, f);
  x = with_lane_xor<8>(x, f);
  x = with_lane_xor<4>(x, f);
  x = with_lane_xor<2>(x, f);
  return with_lane_xor<1>(x, f);
}

// Sum over the 64 lanes of a wavefront; every lane gets the total.
__device__ __forceinline__ float wave_sum(float x) {
  return __uint_as_float(wave_combine(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(__uint_as_float(a) + __uint_as_float(b));
  }));
}

__device__ __forceinline__ float wave_max(float x) {
  return __uint_as_float(wave_combine(__float_as_uint(x), [](uint32_t a, uint32_t b) {
    return __float_as_uint(fmaxf(__uint_as_float(a), __uint_as_float(b)));
  }));
}

__device__ __forceinline__ int wave_min_int(int x) {
  return (int)wave_combine((uint32_t)x, [](uint32_t a, uint32_t b) { return (uint32_t)((int)a < (int)b ? (int)a : (int)b); });
}

// Adds the squares of the 8 bf16 values in q: low halves into acc0, high halves into acc1.  The
// RMS statistic of every kernel goes through this (and wave_sum) so that all of them get the
// same bits for the same row.
__device__ __forceinline__ void accum_sq(const uint4 q, float& acc0, float& acc1) {
  const uint32_t w[4] = {q.x, q.y, q.z, q.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float lo = bf16_lo(w[i]), hi = bf16_hi(w[i]);
    acc0 = fmaf(lo, lo, acc0);
    acc1 = fmaf(hi, hi, acc1);
  }
}

__device__ __forceinline__ float inv_rms_from_sumsq(float ss, int d, float eps) {
  return 1.0f / sqrtf(ss / (float)d + eps);
}

}  // namespace ll
