// Single-precision products on the fp16 matrix cores: a number, taken times a power of two, as the sum of two fp16 terms.
#pragma once
#include "common.hpp"

namespace spdl {

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef unsigned u32x2 __attribute__((ext_vector_type(2)));
typedef float acc32x32 __attribute__((ext_vector_type(16)));

// Powers of two, as exponents of fp32 (127: one), that bring the largest number of a row or a column to 2^12 .. 2^13; the
// number from which on another one is needed, 2^15 after scaling.  (Numbers from 2^125 on, infinities: the smallest one, whose limit is infinity.
// Nothing seen yet: kNoScale, with limit 0.)
constexpr int kNoScale = 254;
constexpr float kLowScale = 2048.f;      // the low terms are taken times this: as far from fp16's smallest exponent as the high ones
__device__ __forceinline__ int scale_for(float largest) {
  return max(14, min(254, 266 - (int)(__builtin_bit_cast(unsigned, largest) >> 23)));
}
__device__ __forceinline__ float scale_limit(int scale) { return __builtin_bit_cast(float, (269 - scale) << 23); }

// What a power of two of a whole row or column costs: a scaled number below 2^-13 is held to 2^-36, not to 2^-23 of itself, so that a product may be
// off by 2^-21 (2^-36 times 2^15; half as much again where low low is left out), however small it is.  The largest number need not be one that
// the sum has a use for: it may be multiplied by a zero.  A scaled sum of `count` products, or with as many among them that may be off
// (scaled_loses), is therefore taken only if it is no smaller than this.  What is lost is then no more than 8 sqrt(count) 2^-24 of the sum of absolute products, if all of it has one sign, and 5 x 2^-24 as a
// root of the mean square (1.5 times that without low low); fp32 roundings of so many terms come to sqrt(count) 2^-24.  Any other sum is
// computed again without the matrix cores.  (Sums of normally distributed numbers are some sqrt(count) 2^22.4: one in seven million is below it.
// 8192 x 10240 at 30 %, n = 128, has a million sums, and one that is gathered makes it 6 us slower: 2.7 % with eight times as much, 0.4 % here.)
__device__ __forceinline__ float scaled_floor(int count) { return __builtin_sqrtf((float)count); }
// Whether a number of a row or a column in whose scaled numbers one is `unit` is among those, below 2^-13 and not zero, that lose bits: as many
// products as there are such numbers in the two may be off, and where there are none, as between whole numbers, a sum may be
// as small as it likes.
__device__ __forceinline__ bool scaled_loses(float x, float unit) {
  return __builtin_bit_cast(unsigned, __builtin_fabsf(x)) - 1u < __builtin_bit_cast(unsigned, unit * 0x1p-13f) - 1u;
}

// Two numbers times `times`: the high terms, and what is left of them, times kLowScale, as the low ones.
__device__ __forceinline__ void split_f16(float x0, float x1, float times, f16x2& high, f16x2& low) {
  high = __builtin_convertvector((f32x2{x0 * times, x1 * times}), f16x2);
  const f32x2 rest = {__builtin_fmaf(x0, times, -(float)high[0]), __builtin_fmaf(x1, times, -(float)high[1])};
  low = __builtin_convertvector((f32x2{rest[0] * kLowScale, rest[1] * kLowScale}), f16x2);
}

__device__ __forceinline__ acc32x32 mfma_f16(f16x8 a, f16x8 b, acc32x32 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0);
}

// The larger of a lane's number, zero or more, and that of the lane 32 on, in both.
__device__ __forceinline__ float max_of_halves(float x) {
  const u32x2 both = __builtin_amdgcn_permlane32_swap(__builtin_bit_cast(unsigned, x), __builtin_bit_cast(unsigned, x), false, false);
  const unsigned low = both[0], high = both[1];          // (a bit cast of both[1] itself reads the first element)
  return __builtin_bit_cast(float, low > high ? low : high);
}

__device__ __forceinline__ bool split_failed(float v) { return !(__builtin_fabsf(v) < __builtin_inff()); }

}  // namespace spdl
