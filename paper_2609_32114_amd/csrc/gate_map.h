// gate_map.h -- raw gate projection -> log-gate, -softplus(x).
//
// -softplus(x) = -(max(x, 0) + log1p(e^-|x|)), the form in which the exponential
// cannot overflow.  Both functions are polynomials whose first terms are taken
// in fp64 and whose tails, small beside them, in fp32; the sum is rounded to
// fp32 once.  Largest error over 2.9 million points of every binade: 0.72 ulp, in
// subnormal results 0.52 (log1pf(expf()) with correctly rounded functions 1.45;
// an earlier form in fp32 throughout 3.7, and 0 for subnormal results).  KDA maps
// a gate per channel and decode one per state row and lane, so its cost shows: a
// decode step of 45 raw KDA sequences 19.0 us with this form or the fp32 one, 20.4
// with every term in fp64; six raw KDA sequences at d = 64 90.5, 89.6 and 91.3.
// Only IEEE operations, so host and device agree bit for bit.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace hagdn {

__host__ __device__ __forceinline__ float neg_softplus(float x) {
  // e^a, a = -|x|: below -110 it is under half the least subnormal fp32 (a NaN
  // stays out of the exponential and comes back through the maximum)
  const float a = __builtin_fmaxf(-__builtin_fabsf(x), -110.f);
  // e^a = 2^n 2^f, |f| <= 1/2 + 2^-17; 2^f by its polynomial through the degree 6
  // Chebyshev nodes (relative error 2^-28.5)
  const float n = __builtin_rintf(a * 1.44269504f);
  const double f = __builtin_fma((double)a, 1.4426950408889634, -(double)n);
  const float g = (float)f;
  float u = 0.00015461444698569338f;
  u = __builtin_fmaf(u, g, 0.001340042817761594f);
  u = __builtin_fmaf(u, g, 0.009618056678524637f);
  u = __builtin_fmaf(u, g, 0.05550327226670302f);
  double p = __builtin_fma((double)u, f, 0.24022650922288757);
  p = __builtin_fma(p, f, 0.6931472067028326);
  p = __builtin_fma(p, f, 1.0);
  const double e = __builtin_bit_cast(double, __builtin_bit_cast(uint64_t, p) + ((uint64_t)(int64_t)(int)n << 52));
  // log1p(e) / e on [0, 1], through the degree 10 Chebyshev nodes (2^-30.1)
  const float h = (float)e;
  float v = 0.001986696593659383f;
  v = __builtin_fmaf(v, h, -0.013187826565608716f);
  v = __builtin_fmaf(v, h, 0.04100657369402377f);
  v = __builtin_fmaf(v, h, -0.08188040923590549f);
  v = __builtin_fmaf(v, h, 0.12377995867876915f);
  v = __builtin_fmaf(v, h, -0.16087623009298038f);
  v = __builtin_fmaf(v, h, 0.19885820285009045f);
  double q = __builtin_fma((double)v, e, -0.24986496459410015);
  q = __builtin_fma(q, e, 0.33332497543526524);
  q = __builtin_fma(q, e, -0.4999997949139123);
  q = __builtin_fma(q, e, 0.9999999991556823);
  return -(float)__builtin_fma(e, q, x < 0.f ? 0.0 : (double)x);
}

}  // namespace hagdn
