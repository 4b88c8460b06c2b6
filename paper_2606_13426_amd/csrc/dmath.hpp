// Float64 normal-CDF primitives for the acceptance scan and U-sampling,
// written in log space as App. A.2 of the paper recommends.
//
// Every function here takes one instruction path for every argument: the
// U-sampler evaluates them on all 64 lanes of a wavefront at points that
// span many orders of magnitude, and a branch on the argument would make the
// wavefront execute every side of it.  Case distinctions are selects between
// values computed on all lanes.
#pragma once

#include <hip/hip_runtime.h>
#include <math.h>

#include "erfcx_table.hpp"

namespace sd {

constexpr double kSqrt1_2 = 0.70710678118654752440;
constexpr double kInvSqrtPi = 0.56418958354775628695;

// erfcx(y) = e^{y^2} erfc(y) for y >= 0 by Weideman's rational approximation
// (SIAM J. Numer. Anal. 31 (1994)): with Z = (L - y)/(L + y),
//   erfcx(y) = 2 p(Z)/(L + y)^2 + 1/(sqrt(pi) (L + y)),
// p of degree N - 1 (N = 40, coefficients in erfcx_table.hpp; relative error
// below 1e-15 on y >= 0, and y -> infinity gives the 1/(sqrt(pi) y) tail).
__device__ inline double erfcx_pos(double y) {
  const double inv = 1.0 / (kWeidemanL + y);
  const double z = (kWeidemanL - y) * inv;
  // four chains in z^4 instead of one of forty dependent steps in z
  static_assert(kWeidemanN % 4 == 0, "four chains of the same length");
  const double z2 = z * z, z4 = z2 * z2;
  double q[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) q[j] = kWeidemanA[j];
#pragma unroll
  for (int n = 4; n < kWeidemanN; ++n) q[n & 3] = fma(q[n & 3], z4, kWeidemanA[n]);
  const double p = fma(fma(q[0], z, q[1]), z2, fma(q[2], z, q[3]));
  return fma(2.0 * p, inv, kInvSqrtPi) * inv;
}

// The mass below x of the unnormalised residual law (Alg. 7),
//   alpha Phi(x) - Phi(x - v),  x <= u* = log(alpha)/v + v/2, v > 0,
// from e1 = erfcx(|x|/sqrt 2), e2 = erfcx((v - x)/sqrt 2) (v - x >= v/2 > 0)
// and the density ratio E = phi(x - v) / (alpha phi(x)) = e^{v (x - u*)} <= 1:
//   x <= 0: alpha e^{-x^2/2} (e1 - e2 E) / 2   (the common factor e^{-x^2/2}
//           stands outside, so the digits survive far into the left tail),
//   x > 0:  alpha (1 - e^{-x^2/2} (e1 + e2 E) / 2).
// Three transcendentals in all: a sum of logs of the two CDFs with log1p and
// expm1 takes six and is no more accurate (both lose the digits of e1 - e2 E
// when v is small).
//
// mass_terms returns the factor in brackets (with the 1/2) and x^2/2.
__device__ inline double mass_terms(double x, double la, double v, double* hx2) {
  const double us = la / v + 0.5 * v;
  const double e1 = erfcx_pos(fabs(x) * kSqrt1_2);
  const double e2 = erfcx_pos((v - x) * kSqrt1_2) * exp(fmin(v * (x - us), 0.0));
  *hx2 = 0.5 * x * x;
  return fmax(x <= 0.0 ? 0.5 * (e1 - e2) : fma(-0.5 * exp(-*hx2), e1 + e2, 1.0), 0.0);
}

// log(alpha Phi(x) - Phi(x - v)).
__device__ inline double log_excess(double x, double la, double v) {
  double hx2;
  const double m = mass_terms(x, la, v, &hx2);
  return la + (x <= 0.0 ? -hx2 : 0.0) + log(m);
}

// h_j of block verification for j < K_b from log alpha_j and ||Delta_{j+1}||:
// h = w/(w + 1 - alpha), w = alpha Phi(u*) - Phi(u* - ||D||), where E = 1.
// alpha = 1 gives h = 1; ||Delta_{j+1}|| = 0 with alpha < 1 gives h = 0.  A w
// that underflows gives 0, far below the smallest coin (2^-25).
__device__ inline double block_h(double la, double vnext) {
  const bool pos = vnext > 0.0;
  const double vs = pos ? vnext : 1.0;
  double hx2;
  const double us = la / vs + 0.5 * vs;
  const double m = mass_terms(us, la, vs, &hx2);
  const double w = m * exp(us <= 0.0 ? la - hx2 : la);
  const double h = w / (w - expm1(la));
  return la >= 0.0 ? 1.0 : pos ? h : 0.0;
}

}  // namespace sd
