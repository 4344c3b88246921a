// GELU(x) = x Phi(x) = max(x, 0) - a Phi(-a) with a = |x|, three ways.
#pragma once
#include <hip/hip_runtime.h>

namespace hmi {

// a Phi(-a) is a smooth bump (at most 0.17, below 1.3e-4 beyond a = 4): Phi(-a) is replaced by a degree-6 polynomial
// Q(a) on [0, 4], fitted so that |a (Q(a) - Phi(-a))| <= 2e-4 everywhere (a is clamped at 4); GELU(0) = 0 exactly.
// Nine fp32 vector-ALU operations (36 clocks a wavefront), no transcendental: for the epilogues of large bf16 launches,
// where the matrix cores wait for it (in u = a / 2 - 1 and with fmaxf eleven; persistent GEMM of 65 536 rows 296 us -> 293, of 177 tenants' 65 536
// 396 -> 390).  (The same polynomial in packed fp16 is 1.5 % of a launch faster, but its rounding
// lifts the error to 5e-4 near x = -3.8, where the result itself is only -2e-4: not used.)
// GELU(+inf) = +inf; a NaN stays one: minimum and maximum hand NaN on, one instruction each (fmaxf takes two).
__device__ __forceinline__ float gelu_poly(float x) {
  const float a = __builtin_elementwise_minimum(fabsf(x), 4.0f);
  float q = -0.00064281153f;
  q = fmaf(q, a, 0.00992081035f);
  q = fmaf(q, a, -0.0575616173f);
  q = fmaf(q, a, 0.139957175f);
  q = fmaf(q, a, -0.0427891985f);
  q = fmaf(q, a, -0.390830964f);
  q = fmaf(q, a, 0.500494301f);
  return fmaf(-a, q, __builtin_elementwise_maximum(x, 0.0f));
}

// Phi(-a) = exp(-a^2 / 2) t P(t), t = 1 / (1 + 0.3 a): exp(a^2 / 2) Phi(-a) is smooth in t, and the degree-7 P was fitted
// (least squares, reweighted towards equal relative errors) to 1.5e-7 relative over [0, 14], beyond which exp underflows.
// For results that are rounded to bf16 behind it: errors of 1e-6 of the value down to x = -4, and small in the negative tail
// too, where 0.5 x (1 + erf(x / sqrt 2)) cancels (2.7e-6 down to -8, 8e-6 to -13, from rounding exp2's argument).
// Fourteen operations and two transcendentals (88 clocks a wavefront; erff takes about twice that).
// What is not finite comes out as x Phi(x) has it: +inf for +inf, NaN for -inf (infinity times zero) and NaN.  Hence a is
// |x| only below 14: above, where nothing is taken off x any more, an infinite a would meet t = 0.
__device__ __forceinline__ float gelu_f32(float x) {
  const float a = __builtin_elementwise_maximum(-x, __builtin_elementwise_minimum(x, 14.0f));   // both hand NaN on
  const float t = __builtin_amdgcn_rcpf(fmaf(0.3f, a, 1.0f));
  float p = 0.03567523509263992f;
  p = fmaf(p, t, -0.15720497071743011f);
  p = fmaf(p, t, 0.2063566893339157f);
  p = fmaf(p, t, -0.053686533123254776f);
  p = fmaf(p, t, 0.12856313586235046f);
  p = fmaf(p, t, 0.09991303831338882f);
  p = fmaf(p, t, 0.12075402587652206f);
  p = fmaf(p, t, 0.11962929368019104f);
  const float e = __builtin_amdgcn_exp2f(a * a * -0.72134752044448170f);   // exp(-a^2 / 2)
  return fmaf(-a * t * p, e, fmaxf(x, 0.0f));
}

// For fp32 results.  Near zero, where the hidden values are, erf's own small error counts where gelu_f32's is that of Phi(-a),
// about one half: over N(0, 0.3) the relative error is 4e-8 here and 9e-8 there (two fp32 encoder layers, 1 728 rows: 672 us for 664).
__device__ __forceinline__ float gelu_erf(float x) { return 0.5f * x * (1.0f + erff(x * 0.70710678118654752f)); }

}  // namespace hmi
