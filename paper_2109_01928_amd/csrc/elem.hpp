// FP64 elementary functions of the target synthesis, for arguments in the
// ranges it meets (the callers check them and take the library's functions
// otherwise).  Each is its argument reduction and a polynomial: Taylor series
// cut where the next term is below a quarter ulp, except the arctangent's,
// which is the Chebyshev interpolant of degree 10.  Errors stay near one ulp.
// Without the library's special cases and its extra-precise logarithm they take
// 36 (log), 27 (exp), 43 (sine and cosine) and 44 (arctangent of a quotient)
// vector instructions where log, exp, sincos and atan2 take 98, 42, 100 and
// 105.  The polynomial's steps are written out with their coefficient in a
// scalar register: the compiler moves a constant addend into vector registers
// before the fused multiply-add (two instructions more), and read from constant
// memory the coefficients' loads are waited for (2,048 tables of 4,096 points
// 299 us against 234, before the pairs below took it to 225-245, by the machine).  Against 80-bit arithmetic the
// relative errors of HN targets are 9.0e-17 (real) and 1.7e-16 (imaginary part)
// rms and 7.5e-16 at most; with the library's functions 9.7e-17, 2.7e-16 and
// 2.5e-15.
#pragma once

#include "common.hpp"

namespace dfit {
namespace elem {

constexpr double LN2_HI = 0x1.62e42fef00000p-1;   // 33 bits of ln 2: n LN2_HI is exact for |n| < 2^20
constexpr double LN2_LO = 0x1.473de6af278edp-34;
constexpr double LOG2E = 0x1.71547652b82fep+0;
constexpr double PI_2_HI = 0x1.921fb54442d18p+0, PI_2_LO = 0x1.1a62633145c07p-54;
constexpr double TWO_PI_INV = 0x1.45f306dc9c883p-1;   // 2 / pi

// coefficients, highest power first
constexpr double LOG_C[10] = {2.0 / 21.0, 2.0 / 19.0, 2.0 / 17.0, 2.0 / 15.0, 2.0 / 13.0, 2.0 / 11.0, 2.0 / 9.0,
                                 2.0 / 7.0, 2.0 / 5.0, 2.0 / 3.0};
constexpr double EXP_C[12] = {1.0 / 6227020800.0, 1.0 / 479001600.0, 1.0 / 39916800.0, 1.0 / 3628800.0,
                                 1.0 / 362880.0, 1.0 / 40320.0, 1.0 / 5040.0, 1.0 / 720.0, 1.0 / 120.0, 1.0 / 24.0,
                                 1.0 / 6.0, 0.5};
constexpr double SIN_C[8] = {1.0 / 355687428096000.0, -1.0 / 1307674368000.0, 1.0 / 6227020800.0,
                                -1.0 / 39916800.0, 1.0 / 362880.0, -1.0 / 5040.0, 1.0 / 120.0, -1.0 / 6.0};
constexpr double COS_C[8] = {1.0 / 20922789888000.0, -1.0 / 87178291200.0, 1.0 / 479001600.0, -1.0 / 3628800.0,
                                1.0 / 40320.0, -1.0 / 720.0, 1.0 / 24.0, -0.5};
constexpr double ATAN_C[11] = {-0x1.3a2b7a07caea9p-6, 0x1.41603647c7a7cp-5, -0x1.a098bb6ba4941p-5,
                                  0x1.dfe61e80903d2p-5, -0x1.10fa75382537fp-4, 0x1.3b1262d95579ep-4,
                                  -0x1.745d0b26b83e7p-4, 0x1.c71c7185314cbp-4, -0x1.24924924360cbp-3,
                                  0x1.999999999934ap-3, -0x1.5555555555555p-2};

template <int K> __device__ __forceinline__ double horner(const double (&c)[K], double x) {
  double p = __builtin_fma(c[0], x, c[1]);
#pragma unroll
  for (int i = 2; i < K; ++i) asm("v_fma_f64 %0, %0, %1, %2" : "+v"(p) : "v"(x), "s"(c[i]));
  return p;
}

// ln x of a normal x > 0: x = m 2^e with m in [sqrt 1/2, sqrt 2), f = m - 1,
// s = f / (2 + f), ln m = 2 atanh s = f - s (f - R) with
// R = 2 (s^2/3 + s^4/5 + ...), s^2 < 0.0295.
// The sum e ln 2 + ln m is returned as a pair hi + lo (lo below an ulp of hi).
struct Pair {
  double hi, lo;
};
__device__ __forceinline__ Pair log_pair(double x) {
  double m = __builtin_amdgcn_frexp_mant(x);
  int e = __builtin_amdgcn_frexp_exp(x);
  const bool low = m < 0x1.6a09e667f3bcdp-1;
  m = low ? m + m : m;
  e = low ? e - 1 : e;
  const double f = m - 1.0;
  const double s = f * rcp_nr(2.0 + f);
  const double z = s * s;
  const double p = horner(LOG_C, z);
  const double de = (double)e;
  const double t = __builtin_fma(de, LN2_LO, -(s * __builtin_fma(-p, z, f)));
  const double h = de * LN2_HI, a = h + f;   // h is exact, and 0 or larger than f
  const double b = t + (f - (a - h));
  const double hi = a + b;
  return {hi, b - (hi - a)};
}
__device__ __forceinline__ double log_pos(double x) { return log_pair(x).hi; }

// e^(c l) for |c l| < 700: c l = x + xl, x = n ln 2 + r, |r| < 0.347.  (With
// the logarithm and the product rounded to doubles, a power's error grows with
// its exponent, to a few ulp; the pair keeps it near one.)
__device__ __forceinline__ double exp_prod(double c, Pair l) {
  const double x = c * l.hi;
  const double xl = __builtin_fma(c, l.lo, __builtin_fma(c, l.hi, -x));
  const double n = rint(x * LOG2E);
  const double r = __builtin_fma(-n, LN2_LO, __builtin_fma(-n, LN2_HI, x) + xl);
  double p = horner(EXP_C, r);
  p = __builtin_fma(p * r, r, r);   // e^r - 1
  return __builtin_amdgcn_ldexp(1.0 + p, (int)n);
}

// sin x and cos x for |x| < 2^20: x = n pi/2 + r, |r| <= pi/4
__device__ __forceinline__ void sincos_mid(double x, double &sn, double &cs) {
  const double n = rint(x * TWO_PI_INV);
  const double r = __builtin_fma(-n, PI_2_LO, __builtin_fma(-n, PI_2_HI, x));
  const double z = r * r;
  const double a = horner(SIN_C, z);
  const double s0 = __builtin_fma(r * z, a, r);
  const double b = horner(COS_C, z);
  const double c0 = __builtin_fma(b, z, 1.0);
  const int q = (int)n;
  const double s1 = (q & 1) ? c0 : s0, c1 = (q & 1) ? s0 : c0;
  sn = (q & 2) ? -s1 : s1;
  cs = ((q + 1) & 2) ? -c1 : c1;
}

// atan(y / x) for x > 0, y >= 0, both well inside the double range: turned by
// 0, pi/4 or pi/2 so that the quotient t has |t| <= tan(pi/8)
__device__ __forceinline__ double atan_quot(double y, double x) {
  constexpr double T = 0x1.a827999fcef32p-2;   // tan(pi/8)
  const bool low = y <= T * x, high = T * y >= x;
  const double num = low ? y : (high ? -x : y - x);
  const double den = low ? x : (high ? y : x + y);
  const double turn = low ? 0.0 : (high ? 2.0 : 1.0);   // in pi/4
  const double r = rcp_nr(den);
  double t = num * r;
  t = __builtin_fma(r, __builtin_fma(-t, den, num), t);
  const double z = t * t;
  const double p = horner(ATAN_C, z);
  const double a = __builtin_fma(t * z, p, t);
  return __builtin_fma(turn, 0.5 * PI_2_HI, __builtin_fma(turn, 0.5 * PI_2_LO, a));
}

}  // namespace elem
}  // namespace dfit
