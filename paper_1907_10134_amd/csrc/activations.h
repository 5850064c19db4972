// tanh and the logistic function in few instructions of short latency, shared by the recurrences (where they sit
// on the dependency chain of every step) and by the kernels that recompute gates.
#pragma once

#include <hip/hip_runtime.h>

// tanh.  Below the seam an odd polynomial, a + a^3 p(a^2), above it 1 - 2 / (e^{2|a|} + 1).  p is the minimax fit
// of (tanh(a) / a - 1) / a^2 on [0, seam], error counted relative to tanh, by Remez exchange in extended
// precision; 2.4e-9 with the coefficients rounded to fp32.  The exponential is taken of a rounded argument x;
// what that rounding left out (lo) and the errors of the sum and of the reciprocal are put right in one
// correction of the reciprocal, so that little but the last rounding remains.  The limit of 40 keeps e finite;
// infinities give 1, NaN stays.
// Largest errors over every second float of [0.5, 4) and 2^18 floats an octave elsewhere, units of 1e-7, those of the
// library's tanhf in brackets; a unit in saturation is exactly 1, its derivative exactly 0 (|a| > 9.1):
//   |a| in                  [0.1, 0.5)    [0.5, 1)      [1, 2)        [2, 4)        [4, 10)
//   tanh, relative          0.62 (0.64)   0.81 (1.48)   0.70 (0.77)   0.35 (0.35)   0.30 (0.30)
//   1 - tanh^2, absolute    0.52 (0.53)   1.17 (1.34)   1.08 (1.15)   0.93 (0.93)   0.89 (0.89)
// One call in a chain of dependent ones takes 50 ns, tanhf 74.
__device__ __forceinline__ float bppsa_tanh(float a) {
  const float u = a * a;
  float p = __builtin_fmaf(-0.000434672955f, u, 0.00252725463f);
  p = __builtin_fmaf(p, u, -0.00820708554f);
  p = __builtin_fmaf(p, u, 0.0216344111f);
  p = __builtin_fmaf(p, u, -0.0539218895f);
  p = __builtin_fmaf(p, u, 0.13332893f);
  p = __builtin_fmaf(p, u, -0.333333194f);
  const float small = __builtin_fmaf(a * u, p, a);
  const float t = __builtin_elementwise_minimum(fabsf(a) + fabsf(a), 40.0f);
  const float x = t * 1.44269504f, lo = __builtin_fmaf(-x, 0.69314718f, t);
  const float e = __builtin_amdgcn_exp2f(x);
  const float r = __builtin_amdgcn_rcpf(e + 1.0f);
  const float left = __builtin_fmaf(-e, r, 1.0f) - r - lo;
  const float big = __builtin_fmaf(-2.0f, __builtin_fmaf(r, left, r), 1.0f);
  return copysignf(fabsf(a) < 0.92f ? small : big, a);
}

// The same without the correction and with the seam at 0.5 (fit on [0, 0.5]: 1.6e-8), for the walk of the tanh RNN
// at H = 20, where every instruction of a step counts: 7 ns a step less than the one above.  Largest relative errors
// in the same units, in brackets those of the form that walk had at first (the same above 0.5, but
// with its seam at 0.1): [0.1, 0.5) 0.64 (11.5), [0.5, 1) 2.3 (2.3), [1, 2) 1.05 (1.05), [2, 4) 0.41 (0.41),
// [4, 10) 0.30 (0.30).
__device__ __forceinline__ float bppsa_tanh_short(float a) {
  const float u = a * a;
  float p = __builtin_fmaf(0.017241491f, u, -0.0530454926f);
  p = __builtin_fmaf(p, u, 0.13325879f);
  p = __builtin_fmaf(p, u, -0.333331436f);
  const float small = __builtin_fmaf(a * u, p, a);
  const float e = __builtin_amdgcn_exp2f(fabsf(a) * 2.88539004f);
  const float big = __builtin_fmaf(-2.0f, __builtin_amdgcn_rcpf(e + 1.0f), 1.0f);
  return copysignf(fabsf(a) < 0.5f ? small : big, a);
}

// 1 / (1 + e^{-a}).  As above the exponential is taken of a rounded argument, and what the rounding left out (lo, to
// second order in ln 2, since it counts in full for a closed gate) and the errors of the sum and of the reciprocal
// are put right in one correction of the reciprocal.  The limits keep infinities out of it: 1 from 88 on, 0 below
// -87.4, where the value is no normal number; NaN stays.  Largest relative errors in units of 1e-7, in
// brackets those of 1 / (1 + expf(-a)):
//   |a| in   [0, 0.1)     [0.1, 0.5)   [0.5, 1)     [1, 2)       [2, 4)       [4, 10)      [10, 20)     [20, 87)
//   a > 0    1.09 (1.09)  1.04 (1.09)  0.96 (1.10)  0.83 (1.02)  0.55 (0.93)  0.34 (0.89)  0.30 (0.61)  0.02 (0.02)
//   a < 0    0.84 (1.28)  0.87 (1.26)  1.11 (1.18)  1.14 (1.29)  1.08 (1.21)  1.08 (1.17)  1.06 (1.48)  1.09 (1.10)
// One call in a chain of dependent ones takes 32 ns, 1 / (1 + expf(-a)) 57.
__device__ __forceinline__ float bppsa_sigmoid(float a) {
  a = __builtin_elementwise_minimum(__builtin_elementwise_maximum(a, -88.0f), 88.0f);
  const float x = a * -1.44269504f;
  const float lo = __builtin_fmaf(-x, -1.90465421e-09f, __builtin_fmaf(-x, 0.693147182f, -a));
  const float e = __builtin_amdgcn_exp2f(x);
  const float r = __builtin_amdgcn_rcpf(1.0f + e);
  const float left = __builtin_fmaf(-(e * r), lo, __builtin_fmaf(-e, r, 1.0f) - r);
  return __builtin_fmaf(r, left, r);
}
