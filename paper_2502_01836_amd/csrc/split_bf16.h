// FP32 operands as three bf16 parts for the bf16 matrix cores: v = v0 + v1 +
// v2, each part the rounded remainder of the ones before (24 bits in all).  A
// product keeps six terms of its parts, x0 w0, x0 w1, x1 w0, x1 w1, x0 w2 and
// x2 w0; the terms left out are 2^-26 of it, below FP32 rounding.  A value
// that rounds to a bf16 infinity has no finite remainder: kernels test the
// magnitudes against kSplitHuge and evaluate such operands in plain FP32.
#pragma once

#include "device_util.h"

namespace leafi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Magnitude bits from which a value rounds to a bf16 infinity (or is one, or a NaN).
constexpr uint32_t kSplitHuge = 0x7f7f8000u;

// Eight FP32 values as three bf16 parts; returns the largest magnitude bits.
__device__ __forceinline__ uint32_t split8(const float (&v)[8], bf16x8 &p0, bf16x8 &p1, bf16x8 &p2) {
  uint32_t big = 0;
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t u = f2u(v[e]) & 0x7fffffffu;
    big = u > big ? u : big;
    p0[e] = static_cast<__bf16>(v[e]);
    const float r1 = v[e] - static_cast<float>(p0[e]);
    p1[e] = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(p1[e]);
    p2[e] = static_cast<__bf16>(r2);
  }
  return big;
}

// Four values into the three planes at element offset `at` of each.
__device__ __forceinline__ uint32_t split_store4(const float4 &v, uint16_t *planes, int plane, int at) {
  const float f[4] = {v.x, v.y, v.z, v.w};
  bf16x4 p0, p1, p2;
  uint32_t big = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t u = f2u(f[e]) & 0x7fffffffu;
    big = u > big ? u : big;
    p0[e] = static_cast<__bf16>(f[e]);
    const float r1 = f[e] - static_cast<float>(p0[e]);
    p1[e] = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(p1[e]);
    p2[e] = static_cast<__bf16>(r2);
  }
  *reinterpret_cast<bf16x4 *>(planes + at) = p0;
  *reinterpret_cast<bf16x4 *>(planes + plane + at) = p1;
  *reinterpret_cast<bf16x4 *>(planes + 2 * plane + at) = p2;
  return big;
}

}  // namespace leafi
