// The nonlinearities of the GRU cell and the output head, one set for every
// kernel whose results have to equal another's bit for bit.
#pragma once

#include <hip/hip_runtime.h>

namespace minsr {

__device__ inline float d_exp(float x) { return expf(x); }
__device__ inline float d_tanh(float x) { return tanhf(x); }
__device__ inline float d_log1p(float x) { return log1pf(x); }
__device__ inline float d_sigmoid(float x) { return 1.f / (1.f + d_exp(-x)); }

// FP64: a cell takes two logistic functions and a tanh per unit, and with the
// library's functions (IEEE division, special cases, tanh in extended
// precision: about 400 instructions a unit) the FP64 kernels are bound by
// their issue.  The ones below reduce x = k ln 2 + r, |r| <= ln 2 / 2 (ln 2 in
// two parts, by fma), take the Taylor polynomial of e^r - 1 to r^13 (remainder
// below 5e-18), and divide by Newton's iteration on the hardware reciprocal:
// about 110 instructions a unit.  Mean and largest error in units in the last
// place over 4e6 arguments against 80-bit values, in brackets the library's:
// exp 0.263, 1.01 (0.256, 0.88); logistic 0.380, 2.38 (0.381, 2.38); tanh
// 0.183, 1.89 (0.161, 0.86); log1p 0.286, 2.12 (0.204, 0.63).  log psi, local
// energies and steps against 64-bit torch keep their errors (10-site FP64
// step: direction 1.8e-14, 2.0e-14 with the library's).  NaN arguments give
// NaN.
__device__ inline double expm1_poly(double r) {
  double p = 1.0 / 6227020800.0;
  p = fma(p, r, 1.0 / 479001600.0);
  p = fma(p, r, 1.0 / 39916800.0);
  p = fma(p, r, 1.0 / 3628800.0);
  p = fma(p, r, 1.0 / 362880.0);
  p = fma(p, r, 1.0 / 40320.0);
  p = fma(p, r, 1.0 / 5040.0);
  p = fma(p, r, 1.0 / 720.0);
  p = fma(p, r, 1.0 / 120.0);
  p = fma(p, r, 1.0 / 24.0);
  p = fma(p, r, 1.0 / 6.0);
  p = fma(p, r, 0.5);
  return fma(p * r, r, r);
}
// x = k ln 2 + r
__device__ inline double reduce_ln2(double x, double& k) {
  k = rint(x * 1.4426950408889634074);
  return fma(-k, 2.3190468138462995584e-17, fma(-k, 0.69314718055994530942, x));
}
// 1 / d for 2^-1000 < |d| < 2^1000
__device__ inline double rcp_newton(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(fma(-d, y, 1.0), y, y);
  return fma(fma(-d, y, 1.0), y, y);
}
// a / (c + b) for c >= |b|: the sum's rounding error goes into the remainder
__device__ inline double quotient(double a, double c, double b) {
  const double d = c + b, dl = b - (d - c);
  const double y = rcp_newton(d), q = a * y;
  return fma(fma(-q, dl, fma(-d, q, a)), y, q);
}
__device__ inline double d_exp(double x) {
  double k;
  // beyond these the result is 0 or infinite
  const double r = reduce_ln2(fmax(fmin(x, 711.0), -746.0), k);
  const double e = ldexp(1.0 + expm1_poly(r), (int)k);
  return x != x ? x : e;
}
__device__ inline double d_tanh(double x) {
  double k;
  const double r = reduce_ln2(fmin(2.0 * fabs(x), 44.0), k);   // tanh(22) rounds to 1
  const double s = ldexp(1.0, (int)k);
  const double e = fma(s, expm1_poly(r), s - 1.0);              // e^2|x| - 1
  const double t = copysign(e > 2.0 ? quotient(e, e, 2.0) : quotient(e, 2.0, e), x);
  return x != x ? x : t;
}
__device__ inline double d_sigmoid(double x) {
  double k;
  const double r = reduce_ln2(fmax(fmin(-x, 708.0), -746.0), k);
  const double e = ldexp(1.0 + expm1_poly(r), (int)k);
  const double t = rcp_newton(1.0 + e);
  return x != x ? x : t;
}
// log(1 + e) for 0 <= e <= 1: 2 atanh(s) with s = f / (2 + f), where 1 + f is
// 1 + e, or (1 + e) / 2 above sqrt(2) - 1, so |s| <= 0.172 and the series to
// s^23 is complete to 1e-19
__device__ inline double d_log1p(double e) {
  const bool big = e > 0.41421356237309504880;
  const double f = big ? 0.5 * (e - 1.0) : e;
  const double s = quotient(f, 2.0, f), z = s * s;
  double p = 2.0 / 23.0;
  p = fma(p, z, 2.0 / 21.0);
  p = fma(p, z, 2.0 / 19.0);
  p = fma(p, z, 2.0 / 17.0);
  p = fma(p, z, 2.0 / 15.0);
  p = fma(p, z, 2.0 / 13.0);
  p = fma(p, z, 2.0 / 11.0);
  p = fma(p, z, 2.0 / 9.0);
  p = fma(p, z, 2.0 / 7.0);
  p = fma(p, z, 2.0 / 5.0);
  p = fma(p, z, 2.0 / 3.0);
  p = fma(p * z, s, s + s);
  return big ? 0.69314718055994530942 + p : p;
}

}  // namespace minsr
