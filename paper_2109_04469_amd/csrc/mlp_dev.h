// Device functions shared by the warm-start network's kernels.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "mlp_internal.h"

namespace pic {

typedef short short8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// FP32 -> BF16, round to nearest even (NaN kept quiet).
__device__ __forceinline__ uint16_t to_bf16(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u && (u & 0x007FFFFFu)) return (uint16_t)((u >> 16) | 0x40u);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ float from_bf16(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

__device__ __forceinline__ float gelu(float z) { return 0.5f * z * (1.0f + erff(z * 0.70710678118654752f)); }
__device__ __forceinline__ float gelu_grad(float z) {
  return 0.5f * (1.0f + erff(z * 0.70710678118654752f)) +
         z * 0.39894228040143268f * expf(-0.5f * z * z);
}

// One parameter's AdamW step from its value w and moments m, v; returns its
// new value.
__device__ __forceinline__ float adam_step(const AdamArgs& a, int64_t i, float gi, float w, float m,
                                           float v) {
  const float mi = a.b1 * m + (1.0f - a.b1) * gi;
  const float vi = a.b2 * v + (1.0f - a.b2) * gi * gi;
  a.m[i] = mi;
  a.v[i] = vi;
  const float mh = mi / a.bc1;
  const float vh = vi / a.bc2;
  const float wn = w - a.lr * (mh / (sqrtf(vh) + a.eps) + a.wd * w);
  a.w[i] = wn;
  return wn;
}

}  // namespace pic
