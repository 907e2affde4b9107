// The channels of one EE pair in FP64 on the vector units: 1/sqrt and 1/(1 + d r) start
// from the hardware estimates and take two Newton steps (about one ulp; FP64 division and
// square root would each expand to a longer correctly-rounded sequence), and the
// polynomials have a compile-time length NQ (coefficients past the true degree are zero).
#pragma once
#include "contract.hpp"

namespace xtc {

template <int NQ>
__device__ __forceinline__ double horner_fixed(const double (&q)[NQ], double x) {
  double r = q[NQ - 1];
#pragma unroll
  for (int j = NQ - 2; j >= 0; --j) r = fma(r, x, q[j]);
  return r;
}

// r = |d| and 1/r (0 and 0 at r = 0, NaN from NaN) from r2 = |d|^2
__device__ __forceinline__ void sqrt_rsqrt(double r2, double& r, double& rinv) {
  double y = __builtin_amdgcn_rsq(r2);            // ~1/sqrt(r2)
  double g = r2 * y, h = 0.5 * y;                  // g ~ sqrt(r2), h ~ 1/(2 sqrt(r2))
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-h, g, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
  }
  const bool zero = r2 == 0.0;
  r = zero ? 0.0 : g;
  rinv = zero ? 0.0 : 2.0 * h;
}

__device__ __forceinline__ double recip(double x) {   // x >= 1
  double y = __builtin_amdgcn_rcp(x);
#pragma unroll
  for (int it = 0; it < 2; ++it) {
    const double e = fma(-x, y, 1.0);
    y = fma(y, e, y);
  }
  return y;
}

}  // namespace xtc
