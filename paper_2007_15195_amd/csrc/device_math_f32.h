// Single-precision normal CDF and quantile pieces for the SOV loop.
//
// The loop works with v = kappa t, kappa = sqrt(log2(e) / 2) (its rows are
// scaled by kappa), so that exp(-t^2/2) = 2^(-v^2).
//
// Phi: with a = |t|, the smaller tail is Phi(-a) = 2^(-v^2) R, where
// R = erfcx(a / sqrt 2) / 2 is a (4,5) rational in |v| fitted by
// fit_fp32_math.py (relative error < 5e-7 in FP32 for a in [0, 40]).
//
// Phi^{-1} below the loop's table: z = -Phi^{-1}(q), q in (0, 1/2], is a (5,4) rational in
// s = sqrt(-log2 q) (relative error < 3.1e-6 in FP32 for s <= 34); where
// log2 q carries an exponent kept outside the FP32 number, a second rational
// covers s in [34, 1100].
//
// Hardware v_log_f32 / v_exp_f32 (base 2), v_sqrt_f32 and v_rcp_f32 are used
// directly; every argument they see is a normal FP32 number or zero.
#pragma once
#include <hip/hip_runtime.h>

#include "fp32_math_coeffs.h"

namespace vecchia {

__device__ __forceinline__ float fast_log2(float x) { return __builtin_amdgcn_logf(x); }
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
__device__ __forceinline__ float fast_rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ float fast_sqrt(float x) { return __builtin_amdgcn_sqrtf(x); }

// The split path's quantile: log2 q carries the exponent kept outside the FP32
// number and reaches -2^20 - 126 (s up to 1025). Up to s = 34 the main rational
// applies; beyond it a (3,2) rational fitted on s in [34, 1100] (relative error
// < 3.3e-7 in FP32) replaces the main one's extrapolation.
__device__ __forceinline__ float ninv_tail_from_log2_split(float lq2) {
  const float s = fast_sqrt(-lq2);
  float p = kZP[5];
#pragma unroll
  for (int c = 4; c >= 0; --c) p = fmaf(p, s, kZP[c]);
  float q = kZQ[4];
#pragma unroll
  for (int c = 3; c >= 0; --c) q = fmaf(q, s, kZQ[c]);
  float z = p * fast_rcp(q);
  if (__builtin_amdgcn_ballot_w64(s > 34.0f) != 0) {   // skipped by waves with no such lane
    float pw = kZPW[3];
#pragma unroll
    for (int c = 2; c >= 0; --c) pw = fmaf(pw, s, kZPW[c]);
    float qw = kZQW[2];
#pragma unroll
    for (int c = 1; c >= 0; --c) qw = fmaf(qw, s, kZQW[c]);
    if (s > 34.0f) z = pw * fast_rcp(qw);
  }
  return z;
}

}  // namespace vecchia
