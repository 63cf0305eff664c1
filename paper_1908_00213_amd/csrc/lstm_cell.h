// The activations of the LSTM cell in the kernels that keep a whole sequence on the device (lstm_seq.hip, lstm_xcd.hip).
#pragma once
#include "common.h"

namespace chn {

// Activations of the cell on the hardware's exponential and reciprocal (relative error a few 1e-7): between two
// exchanges the cell is on the critical path of every step, and the library's expf / tanhf are a third of it.
__device__ __forceinline__ float sigmoid_hw(float x) { return __builtin_amdgcn_rcpf(1.0f + __expf(-x)); }
// tanh: (1 - e) / (1 + e) with e = exp(-2 |x|) cancels for small |x|; there the odd series takes over (its first
// dropped term, 62/2835 x^9, is below 1e-7 of x for |x| < 0.25), so that the relative error stays at a few 1e-7.
__device__ __forceinline__ float tanh_hw(float x) {
  const float ax = fabsf(x), e = __expf(-2.0f * ax);
  const float big = copysignf((1.0f - e) * __builtin_amdgcn_rcpf(1.0f + e), x);
  const float x2 = x * x;
  const float small = x * fmaf(x2, fmaf(x2, fmaf(x2, -17.0f / 315.0f, 2.0f / 15.0f), -1.0f / 3.0f), 1.0f);
  return ax < 0.25f ? small : big;
}

}  // namespace chn
