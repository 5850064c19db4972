// tanh and the logistic function in few instructions of short latency, shared by the recurrences (where they sit
// on the dependency chain of every step) and by the kernels that recompute gates.
#pragma once

#include <hip/hip_runtime.h>

// tanh(a) = a P(a^2) / Q(a^2), both of degree four: the rational minimax approximation of tanh(a) / a on
// [0, 8.3] (relative error 1.2e-8, fitted by linear programming on a grid), evaluated on an argument
// limited to 8, where tanh is 1 to within 2.3e-7.  In fp32 with the hardware's reciprocal: relative error
// 7e-8 rms, 3e-7 at most, over the whole range, no result beyond 1, NaN kept.  It takes as many
// instructions as 1 - 2 / (e^{2a} + 1) with a polynomial for small a, and has half the error.
__device__ __forceinline__ float bppsa_tanh(float a) {
  a = __builtin_elementwise_maximum(__builtin_elementwise_minimum(a, 8.0f), -8.0f);
  const float u = a * a;
  float p = __builtin_fmaf(1.4652938418380183e-08f, u, 2.1511710656341165e-05f);
  float q = __builtin_fmaf(8.296972850985185e-07f, u, 0.00033742646337486804f);
  p = __builtin_fmaf(p, u, 0.0035493590403348207f);
  q = __builtin_fmaf(q, u, 0.026080667972564697f);
  p = __builtin_fmaf(p, u, 0.13426029682159424f);
  q = __builtin_fmaf(q, u, 0.46759355068206787f);
  q = __builtin_fmaf(q, u, 1.0f);
  p = __builtin_fmaf(p, u, 1.0f);
  return a * p * __builtin_amdgcn_rcpf(q);
}

// 1 / (1 + e^{-a}) on the hardware's exponential and reciprocal, the latter refined by one Newton step
// (the minimum keeps an infinite denominator out of it).
__device__ __forceinline__ float bppsa_sigmoid(float a) {
  const float d = 1.0f + __builtin_amdgcn_exp2f(__builtin_elementwise_minimum(a * -1.44269504f, 126.0f));
  const float r = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(__builtin_fmaf(-d, r, 1.0f), r, r);
}
