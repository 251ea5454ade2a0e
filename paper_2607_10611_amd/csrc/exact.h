// Correctly rounded fp32 square root and division for operands of a known
// range, in fewer instructions than the general expansions of sqrtf and `/`.
//
// The step's arithmetic is bound by VALU issue wherever its moments are bf16
// or its weights 4 bits, and two square roots and three divisions are most of
// it.  The general expansions spend half of their instructions on operand
// ranges (v_div_scale twice, v_div_fmas, v_div_fixup; for sqrtf two scalings,
// two neighbours and three selects), at 4 cycles per wave each where an FMA
// takes 2.  Within the ranges below neither is needed.
//
// The square root is one Newton step from the reciprocal root, the division
// Markstein's: a refined reciprocal, the quotient's residual and one correction
// (P. Markstein, Computation of elementary functions on the IBM RISC System/6000
// processor, IBM J. Res. Dev. 34, 1990), with the instruction's approximations to
// start from.  Whether that rounds correctly depends on those, so it is checked
// against the general operations (bench_probes/madd_probes.h): the square root
// and the reciprocal on every fp32 of their ranges, the quotient on every
// denominator significand with 1024 numerators each (madd_check_exact_ops) and,
// by madd_check_quotients, on every pair of significands.
#pragma once

#include <hip/hip_runtime.h>

#include <math.h>
#include <stdint.h>

namespace madd_exact {

constexpr float kTwo64 = 18446744073709551616.0f;  // 2^64
constexpr float kTwoM64 = 1.0f / 18446744073709551616.0f;
constexpr float kTwoM72 = kTwoM64 / 256.0f;
constexpr float kTwo60 = 1152921504606846976.0f;
constexpr float kTwoM60 = 1.0f / 1152921504606846976.0f;
constexpr float kTwoM100 = kTwoM60 / 1099511627776.0f;
constexpr float kTwoM126 = kTwoM64 * kTwoM60 / 4.0f;
constexpr float kTwoM40 = 1.0f / 1099511627776.0f;

// sqrt(x) for x = 0 or a finite x >= 2^-46.  Smaller positive x give at most
// 1.5 sqrt(x); x = -0 gives -0; x <= -2^-71, NaN and Inf give NaN.  The term
// added below the reciprocal root's argument keeps it finite at 0 and is less
// than half a unit in the last place of x from 2^-46 on.
__device__ __forceinline__ float sqrt_in_range(float x) {
  const float y = __builtin_amdgcn_rsqf(x + kTwoM72);
  const float r = x * y, h = 0.5f * y;
  return fmaf(fmaf(-r, r, x), h, r);
}

// 1/d rounded, 2^-126 < |d| < 2^126 (any result for others; NaN for 0 and NaN).
__device__ __forceinline__ float recip_in_range(float d) {
  const float r = __builtin_amdgcn_rcpf(d);
  return fmaf(fmaf(-d, r, 1.0f), r, r);
}

// n/d given r = recip_in_range(d), for a normal quotient, |n| >= 2^-100 (so
// that the residual is exact) or n = +-0, and |n r| < 2^128.  A larger
// quotient gives NaN or Inf, NaN gives NaN; for smaller n the relative error
// stays below 2^-20 or the absolute one below 2^-148 (1 + |r|), with the
// quotient's sign.  The residual is taken with the sign that keeps a zero's.
__device__ __forceinline__ float quot_in_range(float n, float d, float r) {
  const float q = n * r;
  return fmaf(-fmaf(d, q, -n), r, q);
}
__device__ __forceinline__ float div_in_range(float n, float d) {
  return quot_in_range(n, d, recip_in_range(d));
}

// max(|x|, t) as one instruction; a NaN x gives t.
__device__ __forceinline__ float max_abs(float x, float t) {
  float r;
  asm("v_max_f32 %0, |%1|, %2" : "=v"(r) : "v"(x), "v"(t));
  return r;
}

}  // namespace madd_exact
