// Double-precision functions of the (cell, line) setup and the segment laws of
// the march, for the device and (for their tests) the host.
#pragma once

#include <cmath>

#if defined(__HIPCC__)
#include <hip/hip_runtime.h>
#define LRT_HD __host__ __device__ __forceinline__
#else
#define LRT_HD static inline
#endif

namespace lrt {

// 1/x of a normal x: the hardware reciprocal and two Newton steps (five
// instructions against eleven of the correctly rounded division; within an ulp).
// NaN where 1/x overflows (|x| <= 2^-1024) and for infinite x.  The host takes the
// same steps from an estimate as coarse as the hardware's (2^-23).
LRT_HD double rcp_f64(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
#else
    double r = 1.0 / x * (1.0 + 1.1920928955078125e-07);
#endif
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
}
// a/b from rb = rcp_f64(b), refined to the rounding of a division.
LRT_HD double div_f64(double a, double b, double rb)
{
    const double q = a * rb;
    return fma(fma(-b, q, a), rb, q);
}

// e^x = 2^k (1 + p), |x| < 700: k = round(x / ln 2), p = e^r - 1 of the rest r by
// its Taylor series to r^13 (|r| <= ln2/2: the first omitted term is below
// 1.2e-17 of p).  One reduction and one series serve e^x and e^x - 1.
struct ExpParts {
    double p;
    int k;
    double q, r;   // p = r + r^2 q
};
LRT_HD ExpParts exp_parts(double x)
{
    const double kd = rint(x * 1.4426950408889634);
    // ln 2 as a sum of two doubles; the first product is exact inside the fma
    const double r = fma(kd, -2.3190468138462996e-17, fma(kd, -0.6931471805599453, x));
    double q = 1.0 / 6227020800.0;
    q = fma(q, r, 1.0 / 479001600.0);
    q = fma(q, r, 1.0 / 39916800.0);
    q = fma(q, r, 1.0 / 3628800.0);
    q = fma(q, r, 1.0 / 362880.0);
    q = fma(q, r, 1.0 / 40320.0);
    q = fma(q, r, 1.0 / 5040.0);
    q = fma(q, r, 1.0 / 720.0);
    q = fma(q, r, 1.0 / 120.0);
    q = fma(q, r, 1.0 / 24.0);
    q = fma(q, r, 1.0 / 6.0);
    q = fma(q, r, 0.5);
    return ExpParts{fma(q, r * r, r), (int)kd, q, r};
}
LRT_HD double exp_of(const ExpParts &e) { return ldexp(1.0 + e.p, e.k); }
LRT_HD double expm1_of(const ExpParts &e)
{
    const double s = ldexp(1.0, e.k);
    return fma(s, e.p, s - 1.0);
}
// The same for any x: 0, infinity or -1 where the value is out of range, NaN for NaN.
LRT_HD double exp_any(double x) { return exp_of(exp_parts(x < -1e5 ? -1e5 : x > 1e5 ? 1e5 : x)); }
LRT_HD double expm1_any(double x)
{
    const ExpParts e = exp_parts(x < -1e5 ? -1e5 : x > 1e5 ? 1e5 : x);
    return e.k > 60 ? exp_of(e) : expm1_of(e);   // beyond 2^53 the 1 is lost anyway
}

// Laws of a cell-constant and of a linear-j segment of optical depth t (Sec.
// 2.2.3), with f = (1 - e^-t)/t: em = e^-t - 1 and f; e = e^-t and the weights
// per unit length of the near node, (1 - f)/t, and of the far one, (f - e)/t.
// One exponential series and one reciprocal (refined to the rounding of a
// division) per point, 45 instructions, where a library's expm1, exp and
// divisions take 110.  The reciprocal serves only depths of 0.34 to 700.  Below,
// down to zero, subnormals and their signs, the quotients are the series' own:
// with e^-t = 1 + r + r^2 q and r = -t, f is 1 + r q, the near weight q and the
// far one f - q.  Above, up to infinity, there is the plain division.
struct CellLaw {
    double em, f;
};
LRT_HD CellLaw cell_law(double t)
{
    if (!(fabs(t) < 700.0)) {
        const double em = expm1_any(-t);
        return CellLaw{em, -em / t};
    }
    const ExpParts x = exp_parts(-t);
    const double em = expm1_of(x);
    return CellLaw{em, x.k == 0 ? fma(x.q, x.r, 1.0) : div_f64(-em, t, rcp_f64(t))};
}

struct LinearLaw {
    double e, near, far;
};
LRT_HD LinearLaw linear_law(double t)
{
    if (!(fabs(t) < 700.0)) {
        const double f = -expm1_any(-t) / t, e = exp_any(-t);
        return LinearLaw{e, (1.0 - f) / t, (f - e) / t};
    }
    // (e from its own parts: 1 + em keeps no digits of it from t = 37 on)
    const ExpParts x = exp_parts(-t);
    const double s = ldexp(1.0, x.k), e = fma(s, x.p, s);
    if (x.k == 0) return LinearLaw{e, x.q, fma(x.q, x.r, 1.0) - x.q};
    const double em = fma(s, x.p, s - 1.0), rt = rcp_f64(t), f = div_f64(-em, t, rt);
    return LinearLaw{e, div_f64(1.0 - f, t, rt), div_f64(f - e, t, rt)};
}

// Voigt HWHM of the Olivero-Longbothum fit (Sec. 2.2.1) from the Lorentz and
// Doppler ones and 1/(gL + gG): with d = (gL - gG)/(gL + gG),
//   gV/(gL + gG) = 1 - 0.18121 (1 - d^2) - (0.023665 e^{0.6d} + 0.00418 e^{-1.9d}) sin(pi d),
// whose last term is (1 - d^2) h(d) with h entire: its Chebyshev series on
// [-1, 1] to degree 18, as a polynomial (within 4e-17 of h; 19 fused
// multiply-adds in place of two exponentials and a sine, over 100 instructions).
LRT_HD double voigt_hwhm(double gL, double gG, double inv_sum)
{
    constexpr double c[19] = {
        8.027757597623837e-18, 0.08747764743920752, 0.019656945233509734, -0.019332070282700994,
        -0.02501288671355334, -0.0017934143835840583, 0.008573024534664832, 9.676251047635627e-05,
        -0.0010443257874411893, 6.015429973397878e-05, 3.299306941013378e-05, -5.310448664732779e-07,
        2.1131660651870558e-06, -8.610974099941169e-07, -1.29435383230499e-07, 6.996178878525358e-08,
        -1.9832963907340953e-09, -1.86941728690707e-09, 2.428459372221809e-10};
    const double sum = gL + gG, d = (gL - gG) * inv_sum;
    double h = c[18];
#if defined(__HIPCC__)
#pragma unroll
#endif
    for (int i = 17; i >= 0; --i) h = fma(h, d, c[i]);
    return fma(-fma(-d, d, 1.0) * (0.18121 + h), sum, sum);
}

}  // namespace lrt
