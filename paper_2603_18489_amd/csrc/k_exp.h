// The exponential of the vocabulary reduction.  Nothing in here needs the GPU: a test builds this file for the CPU, with a
// rounded 2^t in the hardware instruction's place.
#pragma once
#include <math.h>

namespace ec {

// e^d for -200 <= d <= 0, to about an ulp where that is a normal number: 2^t for the rounded product t = d log2 e, times
// 1 + (d - t ln 2).  float32's ln 2 is 1.9e-9 too large: ln 2 = 0.693147182464600 - 1.9046543e-9.  On MI355X, against 64 bits
// over 2^20 arguments from -87 to -50 as from -9 to -5: 1.4e-7 at most, -3.4e-9 on average, the bias of the hardware's 2^t itself
// (expf: 8.2e-8, -2.4e-9).  Sums of these and of expf's are equally exact: confidences of 5120 rows each of six vocabularies are
// 5.0e-8 to 7.9e-8 off r.m.s. with either.
__device__ __forceinline__ float exp_of_negative(float d) {
  const float t = d * 1.44269502f;
  const float r = fmaf(t, 1.9046543e-9f, fmaf(t, -0.693147182f, d));
  const float e = __builtin_amdgcn_exp2f(t);
  return fmaf(e, r, e);
}

}  // namespace ec
