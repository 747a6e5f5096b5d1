// Exact conversions between binary16 and binary64 for the device kernels that decide codes in
// fp64 (the encoder, the k-means codebook and the fake quantisation).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

__device__ __forceinline__ double h2d(uint16_t b) { return (double)(float)__builtin_bit_cast(_Float16, b); }

// fp64 -> fp16 bits, round to nearest with ties to even, in two steps that round once: to fp32 by
// "round to odd" (toward zero, the last bit set if anything was cut off; 24 bits are more than the
// 11 + 2 that makes the second rounding see every tie and every side of it), then to nearest.
__device__ __forceinline__ uint16_t d2h(double x) {
  const float f = (float)x;
  uint32_t b = __builtin_bit_cast(uint32_t, f);
  const double g = (double)f;
  if (g != x) b = (b - (fabs(g) > fabs(x) ? 1u : 0u)) | 1u;
  return __builtin_bit_cast(uint16_t, (_Float16)__builtin_bit_cast(float, b));
}
