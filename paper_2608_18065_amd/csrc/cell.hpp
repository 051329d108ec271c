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
// two parts, the first of 32 bits so that k times it is exact; r carries its
// rounding error c), take the Taylor polynomial of e^r - 1 to r^13 (remainder
// below 5e-18), and divide by Newton's iteration on the hardware reciprocal,
// the leading sums and quotients with their rounding errors carried: about
// 130 instructions a unit.  Mean and largest error in units in the last place
// over 4e6 arguments against 80-bit values, in brackets the library's: exp
// 0.249, 0.64 (0.256, 0.88); logistic 0.390, 2.36 (0.393, 2.36); tanh 0.203,
// 0.83 (0.205, 0.86); log1p 0.249, 0.63 (0.252, 0.64).  NaN arguments give NaN.
//
// A chain's site waits for every dependent instruction here, so a NaN, a
// quotient's correction and a scale lie beside the chain where they can.  With
// a second branch for e^x far below zero, a move for NaN at the end and k by
// rounding and conversion: chain of 150, d_h = 32, 300 samples 455 us sampling
// and 389 log psi, now 436 and 372; 6 x 6, d_h = 16, 64 samples log psi 104,
// now 101.

// e^r - 1 = r + t, x = k ln 2 + r; t holds r's rounding error too.  x is within
// some limits, which drop a NaN: nan says that it was one, and t is then NaN
// (put back at c, which nothing waits for; a move at the end of a function
// lay in the chain of every site)
__device__ inline void exp_parts(double x, bool nan, int& k, double& r, double& t) {
  const double kb = fma(x, 1.4426950408889634074, 0x1.8p52), kd = kb - 0x1.8p52;
  k = (int)(uint32_t)__builtin_bit_cast(uint64_t, kb);    // the sum's last word is the integer
  const double x1 = fma(-kd, 0x1.62e42feep-1, x);      // exact
  const double l2 = 1.9082149292705877e-10;             // the rest of ln 2
  r = fma(-kd, l2, x1);
  const uint64_t c0 = __builtin_bit_cast(uint64_t, fma(-kd, l2, x1 - r));
  const uint32_t ch = nan ? 0x7FF80000u : (uint32_t)(c0 >> 32);   // (one move: the leading word)
  const double c = __builtin_bit_cast(double, (uint64_t)ch << 32 | (uint32_t)c0);
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
  t = fma(0.5 * r, r, fma(r * r, r * p, c));
}
// 1 / d for 2^-1021 <= |d| < 2^1022
__device__ inline double rcp_newton(double d) {
  double y = __builtin_amdgcn_rcp(d);
  y = fma(fma(-d, y, 1.0), y, y);
  return fma(fma(-d, y, 1.0), y, y);
}
// e^x = m 2^k for x within -746 and 746 (at which it is 0 or infinite)
__device__ inline double exp_mantissa(double x, int& k) {
  double r, t;
  exp_parts(fmax(fmin(x, 746.0), -746.0), x != x, k, r, t);
  const double s = 1.0 + r, lo = r - (s - 1.0);
  return s + (lo + t);
}
__device__ inline double d_exp(double x) {
  int k;
  const double m = exp_mantissa(x, k);
  return ldexp(m, k);
}
__device__ inline double d_tanh(double x) {
  int k;
  double r, t;
  exp_parts(fmin(2.0 * fabs(x), 44.0), x != x, k, r, t);        // tanh(22) rounds to 1
  // e^2|x| - 1 = h + l
  const double s = ldexp(1.0, k), a = s - 1.0, b = fma(s, r, a);
  const double v = fma(s, t, fma(s, r, a - b));
  const double h = b + v, l = v - (h - b);
  // (h + l) / (h + l + 2)
  const double c = fmax(h, 2.0), d = h + 2.0, dl = (fmin(h, 2.0) - (d - c)) + l;
  const double y = rcp_newton(d), q = h * y;
  return copysign(fma(fma(-q, d, h) + fma(-q, dl, l), y, q), x);
}
// (e^-x = m 2^k past the reciprocal's range: that of m 2^1021, scaled)
__device__ inline double d_sigmoid(double x) {
  int k;
  const double m = exp_mantissa(-x, k);
  const int kr = k < 1021 ? k : 1021;
  return ldexp(rcp_newton(1.0 + ldexp(m, kr)), kr - k);
}
// log(1 + e) for 0 <= e <= 1: with 1 + f = 1 + e, or (1 + e) / 2 from e = 1/2
// (both exact), and s = f / (2 + f), |s| <= 0.2, log(1 + f) = 2 atanh(s) =
// f - (f^2 / 2 - s (f^2 / 2 + p)), p = 2 s^2 / 3 + 2 s^4 / 5 + ...; the series
// to s^22 is complete to 1e-18 and takes the quotient q before its correction
__device__ inline double d_log1p(double e) {
  const bool big = e >= 0.5;
  const double f = big ? 0.5 * (e - 1.0) : e;
  const double d = 2.0 + f, dl = f - (d - 2.0), y = rcp_newton(d), q = f * y;
  const double s = fma(fma(-q, dl, fma(-q, d, f)), y, q), z = q * q;
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
  const double g = 0.5 * f, h = g * f, hl = fma(g, f, -h);
  const double l2 = big ? 0.69314718055994530942 : 0.0, l2l = big ? 2.3190468138462995584e-17 : 0.0;
  const double a = l2 + f, al = f - (a - l2);
  const double b = fma(-g, f, a), bl = fma(-g, f, a - b);
  const double u = fma(s, h, fma(s, hl, bl + (al + l2l)));
  return b + fma(s, p * z, u);
}

}  // namespace minsr
