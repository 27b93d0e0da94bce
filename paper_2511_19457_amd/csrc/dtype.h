// Element types of the kernels: raw storage bits and fp32 conversions.
#pragma once

#include <hip/hip_fp16.h>
#include <hip/hip_runtime.h>

#include <cstdint>

#include "sparoa.h"

namespace sparoa {

typedef float f32x2_t __attribute__((ext_vector_type(2)));

template <int DT>
struct Elem;

template <>
struct Elem<SPAROA_F32> {
  using raw = uint32_t;
  static constexpr int size = 4;
  static constexpr raw mag_mask = 0x7FFFFFFFu;   // all bits but the sign
  __device__ static float to_f32(raw v) { return __uint_as_float(v); }
  __device__ static raw from_f32(float v) { return __float_as_uint(v); }
};

template <>
struct Elem<SPAROA_F16> {
  using raw = uint16_t;
  static constexpr int size = 2;
  static constexpr raw mag_mask = 0x7FFFu;
  __device__ static float to_f32(raw v) { return __half2float(__ushort_as_half(v)); }
  __device__ static raw from_f32(float v) { return __half_as_ushort(__float2half_rn(v)); }
  // two elements in one word (one conversion instruction)
  __device__ static uint32_t pack2(float lo, float hi) {
    typedef _Float16 h2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, h2));
  }
};

template <>
struct Elem<SPAROA_BF16> {
  using raw = uint16_t;
  static constexpr int size = 2;
  static constexpr raw mag_mask = 0x7FFFu;
  // bfloat16 is the upper half of a binary32.
  __device__ static float to_f32(raw v) { return __uint_as_float((uint32_t)v << 16); }
  // Round to nearest, ties to even (gfx950 converts in hardware: v_cvt_pk_bf16_f32).
  __device__ static raw from_f32(float f) { return __builtin_bit_cast(raw, (__bf16)f); }
  __device__ static uint32_t pack2(float lo, float hi) {
    typedef __bf16 b2 __attribute__((ext_vector_type(2)));
    return __builtin_bit_cast(uint32_t, __builtin_convertvector(f32x2_t{lo, hi}, b2));
  }
};

// Nonzero elements (magnitude bits set) among 2 W 16-bit floats held in W
// words: a min with 1 in each half, summed by halves.
template <int W>
__device__ __forceinline__ uint32_t nonzeros16(const uint32_t (&w)[W]) {
  typedef uint16_t u16x2 __attribute__((ext_vector_type(2)));
  u16x2 n = u16x2{0, 0};
#pragma unroll
  for (int i = 0; i < W; ++i) {
    const u16x2 m = __builtin_bit_cast(u16x2, w[i] & 0x7FFF7FFFu);
    n += __builtin_elementwise_min(m, u16x2{1, 1});
  }
  return (uint32_t)n.x + (uint32_t)n.y;
}

// relu: max(v, 0); relu6: min(max(v, 0), 6); none: v (a NaN becomes 0 under
// relu and relu6).  Three instructions per element whatever `act` is: early
// returns compile to scalar branches around every element of an unrolled
// epilogue, and compare-and-select forms took five.
__device__ __forceinline__ float apply_act(float v, int act) {
  const float hi = act == SPAROA_ACT_RELU6 ? 6.f : __builtin_inff();
  const float u = __builtin_fminf(__builtin_fmaxf(v, 0.f), hi);
  return act == SPAROA_ACT_NONE ? v : u;
}

}  // namespace sparoa
