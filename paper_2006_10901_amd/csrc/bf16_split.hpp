// Single-precision products on the bf16 matrix cores: a number as the sum of three bf16 terms.
#pragma once
#include "f16_split.hpp"

namespace spdl {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

// x = high + mid + low, each term the rounded rest of the ones before: 3 x 8 bits hold the 24 bits of x
// exactly.  A product of two such numbers is six products of terms (high high; high mid, mid high; mid mid, high
// low, low high); the three left out are below 2^-24 of it.  bf16 products are exact in fp32, and the matrix
// cores add them up in fp32: `sum` takes high high, `rest` the five small ones, so that these are not rounded to
// the large sum's last place one by one.
// The terms of numbers below 2^-102 would lose bits to bf16's smallest exponent, so both operands are taken
// times 2^24 and the result times 2^-48.  Numbers from 2^103 on, or sums from 2^79 on, come out as Inf or NaN
// then, as do infinities and NaN (Inf - Inf): what comes out like that is computed again without the
// matrix cores.
// (Against 64 bits, normally distributed values, 2-norm of the error over that of the result: dot products of 32 / 64 / 128 columns
// 3.9 / 5.0 / 6.5e-8, where the direct kernels have 6.2 / 6.8 / 7.7e-8 and the lane kernel 7.9 / 8.3 / 8.8e-8.  With one accumulator for all
// six: 1.6e-7.)
constexpr float kSplitScale = 16777216.f;                // 2^24
constexpr float kSplitUnscale = 0x1p-48f;

struct Split8 { bf16x8 high, mid, low; };

// Two numbers to bf16 (one instruction), and the rests.
__device__ __forceinline__ unsigned split_term(f32x2& x) {
  const unsigned t = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
  x[0] -= __builtin_bit_cast(float, t << 16);
  x[1] -= __builtin_bit_cast(float, t & 0xffff0000u);
  return t;
}

__device__ __forceinline__ Split8 split8(const float (&v)[8]) {
  u32x4 high, mid, low;
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    f32x2 x = {v[2 * t] * kSplitScale, v[2 * t + 1] * kSplitScale};
    high[t] = split_term(x);
    mid[t] = split_term(x);
    low[t] = __builtin_bit_cast(unsigned, __builtin_convertvector(x, bf16x2));
  }
  return {__builtin_bit_cast(bf16x8, high), __builtin_bit_cast(bf16x8, mid), __builtin_bit_cast(bf16x8, low)};
}

__device__ __forceinline__ acc32x32 mfma_bf16(bf16x8 a, bf16x8 b, acc32x32 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

// Dot product of two rows by one lane, in column order: what the matrix cores cannot give.
__device__ __forceinline__ float split_lane_dot(const float* __restrict__ l, const float* __restrict__ r, int n) {
  float acc = 0.f;
#pragma unroll 1
  for (int j = 0; j < n; ++j) acc = __builtin_fmaf(l[j], r[j], acc);
  return acc;
}

}  // namespace spdl
