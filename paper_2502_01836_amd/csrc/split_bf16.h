// FP32 operands as three bf16 parts for the bf16 matrix cores: v = v0 + v1 +
// v2, each part the rounded remainder of the ones before.  A product keeps six
// terms of its parts, x0 w0, x0 w1, x1 w0, x1 w1, x0 w2 and x2 w0; the terms left
// out are 2^-26 of it, below FP32 rounding.  That holds for operands whose parts
// are exact (all 24 bits, which those below about 2^-110 lose: bf16 ends at
// 2^-133) and whose products cannot overflow in any order of their sum (a sum
// that FP32 takes to +inf could be +inf - inf in parts).  Kernels look at every
// operand they split (SplitRange) and evaluate those out of range in plain
// FP32.
#pragma once

#include "device_util.h"

namespace leafi {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float floatx4 __attribute__((ext_vector_type(4)));

// Magnitude bits from which an operand is out of range: 2^59, so that the sums
// of up to 512 products stay below 2^127 (an infinity and a NaN are above it
// too); and those below which one other than 0 is: 2^-110.
constexpr uint32_t kSplitLarge = 0x5d000000u, kSplitSmall = 0x08800000u;

// Eight FP32 values as three bf16 parts; returns whether one is out of range.
__device__ __forceinline__ bool split8(const float (&v)[8], bf16x8 &p0, bf16x8 &p1, bf16x8 &p2) {
  uint32_t big = 0, small = ~0u;  // (less 1, which puts 0 past every other magnitude)
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const uint32_t u = f2u(v[e]) & 0x7fffffffu;
    big = u > big ? u : big;
    small = u - 1 < small ? u - 1 : small;
    p0[e] = static_cast<__bf16>(v[e]);
    const float r1 = v[e] - static_cast<float>(p0[e]);
    p1[e] = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(p1[e]);
    p2[e] = static_cast<__bf16>(r2);
  }
  return big >= kSplitLarge || small < kSplitSmall - 1;
}

// What split_store4 met: the largest magnitude's bits, and the bits of what the
// second parts left (the third part is that remainder if its low half is zero:
// half an instruction per value, where the smallest magnitude takes one and a half).
struct SplitRange {
  uint32_t big = 0, low = 0;
  __device__ __forceinline__ bool exceeded() const { return big >= kSplitLarge || (low & 0xffffu) != 0; }
};

// Four values into the three planes at element offset `at` of each.
__device__ __forceinline__ void split_store4(const float4 &v, uint16_t *planes, int plane, int at, SplitRange &range) {
  const float f[4] = {v.x, v.y, v.z, v.w};
  bf16x4 p0, p1, p2;
  uint32_t big = 0, low = 0;
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const uint32_t u = f2u(f[e]) & 0x7fffffffu;
    big = u > big ? u : big;
    p0[e] = static_cast<__bf16>(f[e]);
    const float r1 = f[e] - static_cast<float>(p0[e]);
    p1[e] = static_cast<__bf16>(r1);
    const float r2 = r1 - static_cast<float>(p1[e]);
    low |= f2u(r2);
    p2[e] = static_cast<__bf16>(r2);
  }
  *reinterpret_cast<bf16x4 *>(planes + at) = p0;
  *reinterpret_cast<bf16x4 *>(planes + plane + at) = p1;
  *reinterpret_cast<bf16x4 *>(planes + 2 * plane + at) = p2;
  range.big = big > range.big ? big : range.big;
  range.low |= low;
}

}  // namespace leafi
