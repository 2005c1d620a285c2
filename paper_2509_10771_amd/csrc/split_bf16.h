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

// The bf16 matrix instructions cut the low bits of the smaller addends off downwards: a sum of random terms comes out low
// by 7e-9 to 1e-8 of its rms over 16 to 128 contraction indices and by 5e-11 of it per index over more (fp32 matrix
// instructions: below 1e-10), where its random error is 3e-8 (16 indices) to 1e-6 (4096).  One result does not notice,
// but sums over the rows of a minibatch do: the offset has the same sign in every one.  So every other row of a result is
// computed with its sign reversed: odd rows of the operand whose index becomes the result's row are negated by the
// factor of the scaling, and their sums by that of the unscaling.  Their offset is upward, and it cancels in sums over
// rows, to below 1e-10 at every length.  (The last bits of a row depend on the parity of its place for that.  Where a
// layer's inputs hardly differ from row to row, the cut of the third parts' products is common to all rows beyond its
// offset: 4e-8 of the rms in a column's mean for inputs of 20 +- 1, where a single result's error is 2e-7.)
__device__ __forceinline__ float split_scale(int row) { return row & 1 ? -SPLIT_SCALE : SPLIT_SCALE; }
__device__ __forceinline__ float split_unscale(int row) { return row & 1 ? -SPLIT_UNSCALE : SPLIT_UNSCALE; }

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

// Place of a 16-byte unit (eight consecutive contraction indices, group kg, of column c; part 0) among the units of a split
// weight matrix, and the distance to its next part: the layouts of PackJob (kernels.h).
struct PackPlace { long at; int step; };
__device__ __forceinline__ PackPlace pack_place(int kg, int c, int cols, int units) {
  if (units > 0) {                 // blocks of 64 lanes
    const int gate = c / units, j = c - gate * units, per = units >> 3, wave = j / per, tile = (j - wave * per) >> 4;
    const int first = (((kg >> 2) * (per >> 4) + tile) * (cols / units) + gate) * 3;
    return {(long)(first * 8 + wave) * 64 + (kg & 3) * 16 + (j & 15), 8 * 64};
  }
  return {(long)((kg >> 1) * 6 + (kg & 1)) * cols + c, 2 * cols};
}

}  // namespace rslx
