// FP64 sin/cos in revolutions and 1/sqrt of the pair kernels (inter-body sums and
// field evaluation).
#pragma once

#include <hip/hip_runtime.h>

namespace axs {

// sin and cos of 2 pi t in FP64 for |t| < 2^40 revolutions, with a 1024-entry
// table of (cos, sin)(2 pi j / 1024) held in LDS:
//   y = t + 1.5 * 2^42 (one add; the sum has an ulp of 1/1024) rounds t to the
//   nearest multiple j / 1024, and the low word of y is j, which indexes the
//   table; y - 1.5 * 2^42 is j / 1024 exactly, and so is r = t - j / 1024, in
//   [-1/2048, 1/2048];
//   with x = 2 pi r, |x| <= h = pi / 1024: cos x to x^4 (Taylor; the first
//   dropped term below 1.2e-18) and sin x to x^3, with the x^5 term of its
//   Taylor series economised into x and x^3 by the Chebyshev polynomial T5 on
//   [-h, h] (x^5 ~ (5/4) h^2 x^3 - (5/16) h^4 x, error h^5 / 16 there), so the
//   truncation stays below h^5 / 1920 + h^7 / 5040 = 1.5e-16; both as
//   polynomials in r (coefficients times powers of 2 pi);
//   then the angle sum with the table entry.
constexpr int SC_N = 1024;
constexpr double SC_MAGIC = 6597069766656.0;   // 1.5 * 2^42
constexpr double SC_A = 6.283185307179586476925287;
constexpr double SC_H = SC_A / (2 * SC_N);
constexpr double SC_S1 = SC_A * (1.0 - SC_H * SC_H * SC_H * SC_H / 384.0),
                 SC_S3 = SC_A * SC_A * SC_A * (-1.0 / 6.0 + SC_H * SC_H / 96.0);
constexpr double SC_C2 = -SC_A * SC_A / 2.0, SC_C4 = SC_A * SC_A * SC_A * SC_A / 24.0;
__device__ __forceinline__ void sincos_rev_tab(double t, const double2 *tab, double &s, double &c) {
    const double y = t + SC_MAGIC;
    const double r = t - (y - SC_MAGIC);          // exact
    const double r2 = r * r;
    const double sx = r * fma(r2, SC_S3, SC_S1);
    const double cx = fma(r2, fma(r2, SC_C4, SC_C2), 1.0);
    const double2 e = tab[__double2loint(y) & (SC_N - 1)];   // (cos, sin)(2 pi j / 1024)
    s = fma(e.y, cx, e.x * sx);
    c = fma(e.x, cx, -e.y * sx);
}
// sin and cos of 2 pi R' from r2 = R'^2 and u = 1/R': as sincos_rev_tab, with the
// product r2 u rounded to the table's 1/1024 steps inside one FMA,
// y = r2 u + 1.5 * 2^42, and the remainder r = r2 u - J, J = y - 1.5 * 2^42,
// formed by a second FMA, so the remainder carries the product's full precision
// (R' < 2^40 revolutions).
__device__ __forceinline__ void sincos_phase(double r2, double u, double, const double2 *tab, double &s, double &c) {
    const double y = fma(r2, u, SC_MAGIC);
    const double r = fma(r2, u, -(y - SC_MAGIC));
    const double rr = r * r;
    const double sx = r * fma(rr, SC_S3, SC_S1);
    const double cx = fma(rr, fma(rr, SC_C4, SC_C2), 1.0);
    const double2 e = tab[__double2loint(y) & (SC_N - 1)];   // (cos, sin)(2 pi j / 1024)
    s = fma(e.y, cx, e.x * sx);
    c = fma(e.x, cx, -e.y * sx);
}
// 1/sqrt(x) for finite x > 0: the hardware estimate y (relative error up to
// 5.2e-8 measured over 4M arguments; one Newton step leaves 4e-15) corrected
// to second order in e = 1 - x y^2: 1/sqrt(x) = y (1 - e)^(-1/2)
// = y (1 + e/2 + 3 e^2/8 + ...), the first dropped term 5 e^3/16 below 1e-21
__device__ __forceinline__ double rsq(double x) {
    const double y = __builtin_amdgcn_rsq(x);
    const double e = fma(-x * y, y, 1.0);
    return fma(y, e * fma(e, 0.375, 0.5), y);
}

}  // namespace axs
