// sigmoid.h -- 1 / (1 + e^x) in fp64 for the chain of a dense step.  Plain C++
// apart from the reciprocal estimate, so that it can be held to its bound on
// the CPU.
#pragma once

#include <cmath>

namespace asap {

#ifdef __HIP__
#define ASAP_HD __host__ __device__ __forceinline__
#else
#define ASAP_HD inline
#endif

// x = n ln 2 + r with |r| <= ln 2 / 2 (ln 2 in two parts, the published fdlibm
// split: the first has 33 bits, so that n times it is exact), e^r - 1 from its
// Taylor polynomial of degree 13 (remainder below 5e-18) by Estrin's scheme,
// 1 + e^x as a sum of two doubles, so that its rounding does not reach the
// result, and the reciprocal by two Newton steps on rcp's estimate (22 bits or
// more).  About 25 dependent instructions; the library's exp and division took
// about 1000 cycles of a step of 7000 (4 x 600, B = 16).
// Error: e^r - 1 within 2^-53 (its rounding and those of r), 2^n + 1 within half
// an ulp, a last rounding: below 2 ulp in all.  Over 10^6 points each of [-4, 4]
// and [-40, 40] at most 0.9 and 1.7 ulp; 1 / (1 + exp(x)) with the C library 2.0
// and 2.4.
template <class Rcp>
ASAP_HD double inv_1_plus_exp(double x, Rcp rcp) {
  x = x > 700.0 ? 700.0 : x;  // NaN stays NaN; 1 / (1 + e^700) < 1e-304
  x = x < -700.0 ? -700.0 : x;
  const double n = rint(x * 1.4426950408889634);
  const double s = ldexp(1.0, int(n)), a = 1.0 + s;
  const double r = fma(n, -1.9082149292705877e-10, fma(n, -0.69314718036912382, x));
  const double r2 = r * r, r4 = r2 * r2;
  const double p0 = fma(r2, fma(r, 1.0 / 120, 1.0 / 24), fma(r, 1.0 / 6, 0.5));
  const double p1 = fma(r2, fma(r, 1.0 / 362880, 1.0 / 40320), fma(r, 1.0 / 5040, 1.0 / 720));
  const double p2 = fma(r2, fma(r, 1.0 / 6227020800.0, 1.0 / 479001600), fma(r, 1.0 / 39916800, 1.0 / 3628800));
  const double t = fma(r2, fma(r4, fma(r4, p2, p1), p0), r);  // e^r - 1
  const double d = fma(s, t, a), l = fma(s, t, a - d);        // 1 + e^x = d + l
  double q = rcp(d);
  q = fma(q, fma(-d, q, 1.0), q);
  return fma(q, fma(-l, q, fma(-d, q, 1.0)), q);
}

}  // namespace asap
