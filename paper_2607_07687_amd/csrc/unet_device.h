// Device helpers shared by the U-Net kernels: BF16 conversions and MFMA
// operand loads.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/unet.h"

namespace unet {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

__device__ __forceinline__ float bf2f(uint16_t b) { return __uint_as_float(((uint32_t)b) << 16); }
__device__ __forceinline__ uint16_t f2bf(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

// u with the BF16 halves whose gate value is not positive (or NaN) cleared:
// ReLU backward of a pair of gradients.
__device__ __forceinline__ uint32_t gate2(uint32_t u, uint32_t y) {
  const uint32_t lo = (y & 0xFFFFu) - 1u < 0x7F80u ? 0x0000FFFFu : 0u;
  const uint32_t hi = (y >> 16) - 1u < 0x7F80u ? 0xFFFF0000u : 0u;
  return u & (lo | hi);
}

__device__ __forceinline__ bf16x8 ld8(const uint16_t* p) {
  const uint4 v = *reinterpret_cast<const uint4*>(p);
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}
__device__ __forceinline__ bf16x8 zero8() {
  uint4 v = make_uint4(0, 0, 0, 0);
  bf16x8 r;
  __builtin_memcpy(&r, &v, 16);
  return r;
}

}  // namespace unet
