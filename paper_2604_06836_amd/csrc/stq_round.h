// Square root, reciprocal and quotient in a few instructions, correctly rounded where no intermediate under- or overflows.
#pragma once
#include <hip/hip_runtime.h>

#include <cfloat>

namespace stq {

// Newton steps from the hardware's estimates with exact residuals (Markstein, "Computation of elementary functions on the
// IBM RISC System/6000 processor", 1990).  That they end in the correctly rounded result is checked, not assumed, in
// tests/test_short_forms.py: root and reciprocal over every mantissa at every exponent of their ranges on a gfx950; the
// quotient, given a correctly rounded reciprocal, over every operand pair whose quotient lies so close to the middle
// between two floats that the last step could go the other way (solving for the numerators).

// Correctly rounded square root for x = 0 or 2^-96 <= x <= 2^96.
__device__ __forceinline__ float sqrt_rn_safe(float x) {
  const float y = __builtin_amdgcn_rsqf(fmaxf(x, FLT_MIN));  // finite also for x = 0, whose root comes out as 0
  const float s = x * y, h = 0.5f * y;
  return __builtin_fmaf(__builtin_fmaf(-s, s, x), h, s);
}
// Correctly rounded 1/d for 2^-70 <= d <= 2^40.
__device__ __forceinline__ float rcp_rn_safe(float d) {
  const float y = __builtin_amdgcn_rcpf(d);
  return __builtin_fmaf(__builtin_fmaf(-d, y, 1.0f), y, y);
}
// Correctly rounded n/d from y = the correctly rounded 1/d, for n = +0 or 2^-85 <= |n| <= 2^40 and 2^-70 <= d <= 2^40
// (the quotient is then normal and every residual exact).
__host__ __device__ __forceinline__ float div_rn_safe(float n, float d, float y) {
  const float q = n * y;
  return __builtin_fmaf(__builtin_fmaf(-d, q, n), y, q);
}

}  // namespace stq
