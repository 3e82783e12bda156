// Double-precision functions of the (cell, line) setup, for the device and (for
// their tests) the host.
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
LRT_HD double rcp_f64(double x)
{
#if defined(__HIP_DEVICE_COMPILE__)
    double r = __builtin_amdgcn_rcp(x);
    r = fma(fma(-x, r, 1.0), r, r);
    return fma(fma(-x, r, 1.0), r, r);
#else
    return 1.0 / x;
#endif
}

// e^x = 2^k (1 + p), |x| < 700: k = round(x / ln 2), p = e^r - 1 of the rest r by
// its Taylor series to r^13 (|r| <= ln2/2: the first omitted term is below
// 1.2e-17 of p).  One reduction and one series serve e^x and e^x - 1.
struct ExpParts {
    double p;
    int k;
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
    return ExpParts{fma(q, r * r, r), (int)kd};
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
