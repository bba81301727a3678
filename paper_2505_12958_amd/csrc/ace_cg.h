// Coupling coefficients of the real harmonics as compile-time constants,
// shared by the rank kernels of both precisions.
#pragma once
#include <hip/hip_runtime.h>

namespace ap {

// Selection rule of the real coupling coefficients C^{la lb L}_{m1 m2 M}
// (l_a + l_b + L even): the M-type (cosine for M >= 0, sine for M < 0) is the
// product of the m1- and m2-types and |M| is |m1| + |m2| or ||m1| - |m2||.
// Every non-zero entry satisfies it; the library's coefficient table holds
// one value per entry of this superset, in (m1, m2, M) order.
__device__ constexpr int iabs_c(int v) { return v < 0 ? -v : v; }
__device__ constexpr bool cg_rule(int m1, int m2, int M) {
  return ((M < 0) == ((m1 < 0) != (m2 < 0))) &&
         (iabs_c(M) == iabs_c(m1) + iabs_c(m2) || iabs_c(M) == iabs_c(iabs_c(m1) - iabs_c(m2)));
}

// ---- coupling coefficients as compile-time constants
// Complex <j1 m1 j2 m2 | J M> from Racah's closed form and the change of
// basis to the real harmonics (real Y_m = sum_mu U_{m mu} Y^mu with
// U_{0,0} = 1; m > 0: U_{m,m} = (-1)^m/sqrt2, U_{m,-m} = 1/sqrt2; m < 0, k = |m|:
// U_{m,k} = -i(-1)^k/sqrt2, U_{m,-k} = i/sqrt2), evaluated by the compiler.
constexpr double ce_fact(int n) {
  double r = 1.0;
  for (int i = 2; i <= n; ++i) r *= i;
  return r;
}
constexpr double ce_sqrt(double x) {
  if (x <= 0.0) return 0.0;
  double r = x > 1.0 ? x : 1.0;
  for (int i = 0; i < 200; ++i) {
    const double n = 0.5 * (r + x / r);
    if (n == r) break;
    r = n;
  }
  return r;
}
constexpr double ce_cg(int j1, int m1, int j2, int m2, int J, int M) {
  if (m1 + m2 != M || iabs_c(m1) > j1 || iabs_c(m2) > j2 || iabs_c(M) > J) return 0.0;
  if (J < iabs_c(j1 - j2) || J > j1 + j2) return 0.0;
  const double pre = (2 * J + 1) * ce_fact(J + j1 - j2) * ce_fact(J - j1 + j2) * ce_fact(j1 + j2 - J) /
                     ce_fact(j1 + j2 + J + 1) * ce_fact(J + M) * ce_fact(J - M) * ce_fact(j1 - m1) *
                     ce_fact(j1 + m1) * ce_fact(j2 - m2) * ce_fact(j2 + m2);
  double sum = 0.0;
  for (int k = 0; k <= j1 + j2 - J; ++k) {
    const int a0 = k, a1 = j1 + j2 - J - k, a2 = j1 - m1 - k, a3 = j2 + m2 - k, a4 = J - j2 + m1 + k,
              a5 = J - j1 - m2 + k;
    if (a0 < 0 || a1 < 0 || a2 < 0 || a3 < 0 || a4 < 0 || a5 < 0) continue;
    const double den = ce_fact(a0) * ce_fact(a1) * ce_fact(a2) * ce_fact(a3) * ce_fact(a4) * ce_fact(a5);
    sum += ((k & 1) ? -1.0 : 1.0) / den;
  }
  return ce_sqrt(pre) * sum;
}
// U_{m, mu} as (re, im); zero unless mu = +-m
struct ce_c2 { double re, im; };
constexpr ce_c2 ce_u(int m, int mu) {
  const double s = 0.70710678118654752440;
  if (m == 0) return mu == 0 ? ce_c2{1.0, 0.0} : ce_c2{0.0, 0.0};
  if (m > 0) {
    if (mu == m) return ce_c2{(m & 1) ? -s : s, 0.0};
    if (mu == -m) return ce_c2{s, 0.0};
    return ce_c2{0.0, 0.0};
  }
  const int k = -m;
  if (mu == k) return ce_c2{0.0, (k & 1) ? s : -s};
  if (mu == -k) return ce_c2{0.0, s};
  return ce_c2{0.0, 0.0};
}
constexpr ce_c2 ce_mul(ce_c2 a, ce_c2 b) { return ce_c2{a.re * b.re - a.im * b.im, a.re * b.im + a.im * b.re}; }
constexpr ce_c2 ce_conj(ce_c2 a) { return ce_c2{a.re, -a.im}; }
// real coupling coefficient C^{l1 l2 L}_{m1 m2 M}
constexpr double ce_real_cg(int l1, int l2, int L, int m1, int m2, int M) {
  double acc = 0.0;
  const int mu1s[2] = {iabs_c(m1), -iabs_c(m1)};
  const int mu2s[2] = {iabs_c(m2), -iabs_c(m2)};
  for (int a = 0; a < (m1 == 0 ? 1 : 2); ++a)
    for (int b = 0; b < (m2 == 0 ? 1 : 2); ++b) {
      const int mu1 = mu1s[a], mu2 = mu2s[b], mu = mu1 + mu2;
      if (iabs_c(mu) > L) continue;
      const ce_c2 u = ce_mul(ce_mul(ce_u(M, mu), ce_conj(ce_u(m1, mu1))), ce_conj(ce_u(m2, mu2)));
      acc += u.re * ce_cg(l1, mu1, l2, mu2, L, mu);
    }
  return acc;
}

}  // namespace ap
