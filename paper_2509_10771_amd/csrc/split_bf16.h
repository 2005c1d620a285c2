// Splitting fp32 values into three bf16 parts for the bf16 matrix cores (see gemm.hip).
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace rslx {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two values rounded to bf16 (nearest even), x in the low half.
__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  return __builtin_bit_cast(uint32_t, __builtin_convertvector((f32x2){x, y}, bf16x2));
}

// Operands are split after multiplication by 2^16, and a sum of their products is multiplied by 2^-32: the last bit of an
// fp32 value is 2^-149 at the smallest, that of a bf16 value 2^-133, so unscaled values would lose their third part
// below 2^-110 and their second below 2^-118.  Values of 2^111 and above, and sums of 2^96 and above, overflow instead and
// are computed in fp32 (see gemm.hip).
constexpr float SPLIT_SCALE = 65536.0f, SPLIT_UNSCALE = 0x1p-32f;

// x = p0.lo + p1.lo + p2.lo, y = p0.hi + p1.hi + p2.hi: both remainders are exact, and the last one has at most eight
// significant bits, so the three parts together are the value itself (multiples of 2^-133).  Infinities, and values
// that round to infinity, leave NaN in the lower parts.
__device__ __forceinline__ void split_pair(float x, float y, uint32_t& p0, uint32_t& p1, uint32_t& p2) {
  p0 = pack_bf16(x, y);
  x -= __uint_as_float(p0 << 16);
  y -= __uint_as_float(p0 & 0xffff0000u);
  p1 = pack_bf16(x, y);
  x -= __uint_as_float(p1 << 16);
  y -= __uint_as_float(p1 & 0xffff0000u);
  p2 = pack_bf16(x, y);
}

}  // namespace rslx
