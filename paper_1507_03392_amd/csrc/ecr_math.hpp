// ecr_math.hpp -- the binary64 functions of a collision's continuous outcome:
// quotients, roots, exponentials and logarithms whose arguments' ranges are
// known, and Nanbu's scattering angle made of them.  No memory, no lane: the
// file also compiles for the host, where its errors are measured.
#pragma once

#include <math.h>

namespace ecr {

// ---------------------------------------------------------------------------
// Functions for continuous outcomes of a collision (never for a decision,
// which keeps the correctly rounded library operations).  A collision is a
// chain of dependent binary64 operations, and its length in time, not in
// instructions, bounds the step: so no library call where the argument's
// range is known, polynomials evaluated in pairs of terms, and everything in
// one block the compiler can interleave.
// div_cont: the hardware reciprocal (relative error below 2^-22) refined once
// and the quotient corrected by its exact remainder: within an ulp.  b must
// be normal with a normal reciprocal.
// root_cont: s = sqrt x and is = 1 / sqrt x from the hardware reciprocal
// square root by coupled (Goldschmidt) steps on the root and half its
// reciprocal, the root corrected by its exact remainder: both within an ulp
// or so.  x must be in [1e-290, 1e290].
// exp_cont: e^x for |x| < 700: x = n ln2 + r, |r| <= ln2 / 2, the Taylor sum
// through r^13 (truncation below 5e-17) with the rounding of 1 + r made good:
// within an ulp.  expm1_cont: e^x - 1 for x < -0.7 from the same sum, with the
// rounding of the difference made good.
// log1p_cont(x) for x in (-1, 0]: y = 1 + x and its rounding error d = x - (y - 1)
// (exact: Sterbenz), y = m 2^e with m in [sqrt(1/2), sqrt(2)), and
// log m = 2 atanh(s), s = (m - 1)/(m + 1), summed as 2 s sum_k z^k/(2k+1),
// z = s^2 <= 0.0295, through k = 11 (truncation below 2^-60 relative);
// log1p x = e ln2 + log m + d/y.  The quotient s is held in two parts, so that
// what is left is the rounding of the last sums: within 2 ulp.
// ---------------------------------------------------------------------------
constexpr double kLn2Hi = 6.93147180369123816490e-01;  // its low 32 bits zero: n kLn2Hi is exact
constexpr double kLn2Lo = 1.90821492927058770002e-10;

__device__ __forceinline__ double div_cont(double a, double b) {
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = a * r;
  return fma(fma(-b, q, a), r, q);
}

// num / g^3 from g2 = g^2, g and ig = 1 / g, whose error enters the product
// three times: the product's remainder against g2 g makes it good, within an
// ulp or so of the exact quotient.  g2 must be in [1e-150, 1e150].
__device__ __forceinline__ double over_cube(double num, double g2, double g, double ig) {
  const double ig3 = (ig * ig) * ig, q = num * ig3;
  return fma(fma(-q, g2 * g, num), ig3, q);
}

__device__ __forceinline__ void root_cont(double x, double &s, double &is) {
  const double h0 = __builtin_amdgcn_rsq(x);
  double g = x * h0, h = 0.5 * h0;
  double r = fma(-g, h, 0.5);
  g = fma(g, r, g);
  h = fma(h, r, h);
  s = fma(fma(-g, g, x), h, g);
  // the root is final now, so the whole of its product's error is h's
  h = h + h;
  is = fma(h, fma(-s, h, 1.0), h);
}

// e^x = (y + w) 2^n
struct ExpParts {
  double y, w;
  int n;
};
__device__ __forceinline__ ExpParts exp_parts(double x) {
  const double n = rint(x * 1.44269504088896340736);
  const double r = fma(-n, kLn2Lo, fma(-n, kLn2Hi, x));
  const double r2 = r * r, r4 = r2 * r2, r8 = r4 * r4;
  const double p01 = fma(r, 1.0 / 6.0, 0.5), p23 = fma(r, 1.0 / 120.0, 1.0 / 24.0);
  const double p45 = fma(r, 1.0 / 5040.0, 1.0 / 720.0), p67 = fma(r, 1.0 / 362880.0, 1.0 / 40320.0);
  const double p89 = fma(r, 1.0 / 39916800.0, 1.0 / 3628800.0);
  const double pab = fma(r, 1.0 / 6227020800.0, 1.0 / 479001600.0);
  const double lo = fma(r2, p23, p01), mid = fma(r2, p67, p45), hi = fma(r2, pab, p89);
  const double q = fma(r8, hi, fma(r4, mid, lo));
  const double y = 1.0 + r;
  return {y, fma(r2, q, r - (y - 1.0)), (int)n};
}
__device__ __forceinline__ double exp_cont(double x) {
  const ExpParts e = exp_parts(x);
  return ldexp(e.y + e.w, e.n);
}
__device__ __forceinline__ double expm1_cont(double x) {
  const ExpParts e = exp_parts(x);
  const double y = ldexp(e.y, e.n), m = y - 1.0;
  return m + (ldexp(e.w, e.n) + (y - (m + 1.0)));
}

__device__ __forceinline__ double log1p_cont(double x) {
  const double y = 1.0 + x;
  const double d = x - (y - 1.0);
  int e;
  double m = frexp(y, &e);
  const bool low = m < 0.70710678118654752440;
  m = low ? m + m : m;
  e = low ? e - 1 : e;
  const double f = m - 1.0;
  // sv + sl = f / (2 + f), 2 + f = b + bl
  const double b = 2.0 + f, bl = f - (b - 2.0);
  double r = __builtin_amdgcn_rcp(b);
  r = fma(fma(-b, r, 1.0), r, r);
  const double q = f * r, rem = fma(-q, bl, fma(-b, q, f));
  const double sv = fma(rem, r, q), sl = fma(rem, r, q - sv);
  const double z = sv * sv, z2 = z * z, z4 = z2 * z2, z8 = z4 * z4;
  const double p01 = fma(z, 2.0 / 5.0, 2.0 / 3.0), p23 = fma(z, 2.0 / 9.0, 2.0 / 7.0);
  const double p45 = fma(z, 2.0 / 13.0, 2.0 / 11.0), p67 = fma(z, 2.0 / 17.0, 2.0 / 15.0);
  const double p89 = fma(z, 2.0 / 21.0, 2.0 / 19.0);
  const double lo = fma(z2, p23, p01), mid = fma(z2, p67, p45), hi = fma(z2, 2.0 / 23.0, p89);
  const double p = fma(z8, hi, fma(z4, mid, lo));
  const double de = (double)e;
  const double t = fma(sv * z, p, fma(2.0, sl, fma(de, kLn2Lo, div_cont(d, y))));
  return fma(de, kLn2Hi, fma(2.0, sv, t));
}

// ---------------------------------------------------------------------------
// Nanbu: 1 - cos(chi) = -log1p(u expm1(-2A))/A with A(s) from the table
// (ln A linear in s between nodes a and b), A = 1/s below 2^-20, isotropic
// from 8.
// ---------------------------------------------------------------------------
constexpr double kSLo = 9.5367431640625e-07;  // 2^-20: A = 1/s below
constexpr double kSHi = 8.0;                  // isotropic at and above

struct NanbuNode {
  double a, b, fr;
};
__device__ __forceinline__ double nanbu_omc(const NanbuNode &nd, double sv, double u) {
  const double x = fma(nd.fr, nd.b - nd.a, nd.a);
  double iA = exp_cont(-x);  // 1 / A
  iA = sv < kSLo ? sv : iA;
  // for A > 20, exp(-2A) < 5e-18 is below half an ulp of 1, so expm1(-2A)
  // rounds to -1 exactly (most pairs of a cool plasma)
  double em = -1.0;
  if (!(iA < 0.05)) {
    const double t = -2.0 * exp_cont(x);
    em = t < -0.7 ? expm1_cont(t) : expm1(t);
  }
  double omc = -log1p_cont(u * em) * iA;
  omc = sv >= kSHi ? 2.0 * u : omc;
  omc = omc < 0.0 ? 0.0 : omc;
  return omc > 2.0 ? 2.0 : omc;
}

}  // namespace ecr
