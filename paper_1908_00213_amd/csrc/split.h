// Three bfloat16 parts of an fp32 value: what the kernels that multiply fp32 operands on the bfloat16 matrix cores share
// (the products of gemm_split.h, where the scheme and its source are described, and the recurrent layer's of lstm_xcd.hip).
#pragma once
#include "common.h"

namespace chn {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float floatx2 __attribute__((ext_vector_type(2)));

__device__ __forceinline__ uint32_t pack_bf16(float x, float y) {
  const floatx2 v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

// The three parts of two neighbouring values, packed (first value in the low half).
__device__ __forceinline__ void split2(float x, float y, uint32_t &h, uint32_t &m, uint32_t &l) {
  h = pack_bf16(x, y);
  x -= __uint_as_float(h << 16);
  y -= __uint_as_float(h & 0xffff0000u);
  m = pack_bf16(x, y);
  x -= __uint_as_float(m << 16);
  y -= __uint_as_float(m & 0xffff0000u);
  l = pack_bf16(x, y);
}

// Both operands are multiplied by 2^24 before they are split, and the sums by 2^-48 at the end, all exact: the bits of an
// fp32 value are multiples of 2^-149, those of a scaled one of 2^-125, so every part of every value, subnormal ones
// included, is a normal bfloat16 number, whatever else its row holds, and what underflow takes from a product lies below 2^-174 of
// the result's scale.  (Unscaled, 2^-120 beside a 1 kept 14 bits.)  The price is the other end: sums from 2^80 on
// overflow, and whoever uses this multiplies them again on fp32 values.
constexpr float kSplitScale = 0x1p24f;

}  // namespace chn
