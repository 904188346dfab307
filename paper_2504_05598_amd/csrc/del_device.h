// Device helpers shared by the kernel files: operand types, bf16 conversion, streaming loads.
#pragma once
#include "del_kernels.h"

namespace del {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float floatx4;

__device__ __forceinline__ float bf16_bits_to_f32(uint32_t h) { return __uint_as_float(h << 16); }
__device__ __forceinline__ uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// A weight tile is read exactly once per launch, so it is fetched with a non-temporal load (no reuse: keeps the
// stream out of the way of the cached activations).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ uint4 ld_stream(const uint4* p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4*)p);
  return make_uint4(v.x, v.y, v.z, v.w);
}

// Four consecutive values -> 16-bit high parts and the 16-bit remainders (together 16 mantissa bits).
__device__ __forceinline__ void split4(const float* v, uint2& hi, uint2& lo) {
  uint16_t h[4], l[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    h[e] = f32_to_bf16_rne(v[e]);
    l[e] = f32_to_bf16_rne(v[e] - bf16_bits_to_f32(h[e]));
  }
  hi = make_uint2((uint32_t)h[0] | ((uint32_t)h[1] << 16), (uint32_t)h[2] | ((uint32_t)h[3] << 16));
  lo = make_uint2((uint32_t)l[0] | ((uint32_t)l[1] << 16), (uint32_t)l[2] | ((uint32_t)l[3] << 16));
}

}  // namespace del
