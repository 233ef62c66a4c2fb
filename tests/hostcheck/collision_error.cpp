/* Errors of the collision's functions (csrc/ecr_math.hpp) against 80-bit
 * arithmetic, beside those of the same formulas with the library's exp and
 * expm1, IEEE quotients and roots.  The hardware's reciprocal and reciprocal
 * root are modelled as the exact ones off by up to 2^-22.  Prints, per
 * class, the mean and largest error in units in the last place: of the
 * functions, then of the plain formulas. */
#include <math.h>
#include <stdint.h>
#include <stdio.h>
#include <string.h>

#include <algorithm>
#include <cmath>
#include <random>

#define __device__
#define __forceinline__ inline
static double off(double v) {
  uint64_t b;
  memcpy(&b, &v, 8);
  b *= 0x9E3779B97F4A7C15ull;
  b ^= b >> 29;
  return v * (1.0 + ((double)(b >> 11) * 0x1p-52 - 1.0) * 0x1p-22);
}
static double model_rcp(double x) { return off(1.0 / x); }
static double model_rsq(double x) { return off(1.0 / sqrt(x)); }
#define __builtin_amdgcn_rcp model_rcp
#define __builtin_amdgcn_rsq model_rsq
#include "ecr_math.hpp"

static double log1p_plain(double x) {
  const double y = 1.0 + x, d = x - (y - 1.0);
  int e;
  double m = frexp(y, &e);
  if (m < 0.70710678118654752440) {
    m = m + m;
    e -= 1;
  }
  const double f = m - 1.0, sv = f / (2.0 + f), z = sv * sv;
  double p = 2.0 / 23.0;
  for (int k = 21; k >= 3; k -= 2) p = fma(p, z, 2.0 / k);
  const double de = (double)e, lm = fma(sv * z, p, 2.0 * sv);
  return fma(de, ecr::kLn2Hi, lm + fma(de, ecr::kLn2Lo, d / y));
}

struct Error {
  const char *name;
  long n = 0;
  double sum[2] = {0, 0}, top[2] = {0, 0};
  void add(long double t, double here, double plain) {
    const double r = fabs((double)t), ulp = std::nextafter(r, INFINITY) - r;
    const double e[2] = {(double)(fabsl(here - t) / ulp), (double)(fabsl(plain - t) / ulp)};
    ++n;
    for (int k = 0; k < 2; ++k) {
      sum[k] += e[k];
      top[k] = std::max(top[k], e[k]);
    }
  }
  void print() const {
    printf("%s %ld %.5f %.3f %.5f %.3f\n", name, n, sum[0] / n, top[0], sum[1] / n, top[1]);
  }
};

int main() {
  std::mt19937_64 r(5);
  std::uniform_real_distribution<double> U(0, 1);
  std::normal_distribution<double> G(0, 1);
  const int n = 1 << 21;

  Error s{"s"};
  for (int i = 0; i < n; ++i) {
    const double sc = exp(5.0 + 9.0 * U(r)), ux = sc * G(r), uy = sc * G(r), uz = sc * G(r);
    const double amu = 1.66053906660e-27, ma = amu * 39.948, mb = i & 1 ? ma : amu * (1 + 100 * U(r));
    const double Cs = 1e-52 * (0.5 + U(r)), nc = 1e16 * (1 + 50 * U(r)), dt = 1e-9 * (0.1 + 10 * U(r));
    const double qq = (double)((1 + r() % 10) * (1 + r() % 10));
    const double mu = (ma * mb) / (ma + mb), g2 = (ux * ux + uy * uy) + uz * uz;
    double g, ig;
    ecr::root_cont(g2, g, ig);
    const double here = ecr::over_cube((((Cs / (mu * mu)) * (qq * qq)) * nc) * dt, g2, g, ig);
    const double plain = (((Cs * (qq * qq)) * nc) * dt) / ((mu * mu) * (g2 * sqrt(g2)));
    const long double lm = (long double)ma * mb / ((long double)ma + mb);
    const long double l2 = (long double)ux * ux + (long double)uy * uy + (long double)uz * uz;
    s.add((long double)Cs * qq * qq * nc * dt / (lm * lm * l2 * sqrtl(l2)), here, plain);
  }
  s.print();

  // by A; u em below -0.9, where 1 + u em cancels, is a class of its own (the
  // error of u em itself, the same in both)
  Error o[6] = {{"A<0.01"}, {"A<0.35"}, {"A<2"}, {"A<20"}, {"A>=20"}, {"cancelling"}};
  for (int i = 0; i < n; ++i) {
    const double x = i % 4 < 2 ? -4.0 + 14.0 * U(r) : -7.0 + 10.5 * U(r);  // ln A
    double u = ((double)(r() >> 11) + 0.5) * 0x1p-53;
    if (i % 8 == 0) u = ldexp(u, -(int)(r() % 40));
    const double A = exp(x), em = A > 20.0 ? -1.0 : expm1(-2.0 * A);
    const double plain = std::min(-log1p_plain(u * em) / A, 2.0);
    const double here = ecr::nanbu_omc({x, x, 0.0}, 1.0, u);
    const long double la = expl((long double)x), lem = expm1l(-2.0L * la);
    const long double t = std::min(-log1pl(u * lem) / la, 2.0L);
    const int c = u * em < -0.9 ? 5 : A < 0.01 ? 0 : A < 0.35 ? 1 : A < 2.0 ? 2 : A < 20.0 ? 3 : 4;
    o[c].add(t, here, plain);
  }
  for (const Error &e : o) e.print();

  // the binary32-mixed s: against the IEEE quotient
  Error q{"quotient"};
  for (int i = 0; i < n; ++i) {
    const double a = U(r) + 0x1p-60, b = exp(40.0 * (U(r) - 0.5));
    q.add((long double)a / (long double)b, ecr::div_cont(a, b), a / b);
  }
  q.print();
  return 0;
}
