// rt_math.h -- natural logarithms in FP64 for the adjoint's dual-number rates
// and the angle of a flux to an axis for the FP64 transport.
//
// The reverse chemistry linearises every substep through the Hui & Gnedin fits
// of App. E.2 and E.3 themselves (the forward attempts read the table of
// rt_rates.h); the library's logarithms carry extended-precision
// intermediates that cost about twice the instructions of the methods below,
// which stay within about 1.2 ulp (ln) and 1.5 ulp (ln(1 + u)) of the exact
// values.
//
//   ln x: x = 2^e m with m in [sqrt(1/2), sqrt(2)); with f = m - 1 (exact)
//   and s = f / (m + 1), ln m = 2 atanh(s) = 2s + 2s^3/3 + 2s^5/5 + ...,
//   |s| <= 3 - 2 sqrt(2), so the odd series to s^21 leaves a truncation
//   below 2^-55 relative.  Since 2s = f - s f, ln m = f - s (f - 2 z q(z))
//   with z = s^2 and q(z) = 1/3 + z/5 + ... + z^9/21: the rounding of s then
//   enters only through the small term s (...).  q is nested as
//   (1/3)(1 + (3/5) z (1 + (5/7) z (1 + ...))): every addend is 1, an inline
//   operand, and the ratios multiply z from scalar registers instead of ten
//   FP64 constants held in vector registers.  ln x = e ln 2 + ln m with
//   ln 2 split into a 32-bit head and its remainder.
//   ln(1 + u): w = 1 + u rounded, c = u - (w - 1) its rounding error (exact
//   for u >= 0), ln(1 + u) = ln w + c / w to first order in c, with 1/w
//   from the reduced mantissa (no second division).
//
// Written with explicit fma() and no other multiply feeding an add, so the
// same source gives the same bits compiled for the host (where its accuracy
// is tested against extended precision) and for the device.
#pragma once
#include <math.h>

namespace rtm1 {

constexpr double RM_LN2_HI = 6.93147180369123816490e-01;  // ln 2 to 32 significant bits
constexpr double RM_LN2_LO = 1.90821492927058770002e-10;  // ln 2 - RM_LN2_HI
constexpr double RM_SQRT_HALF = 0.70710678118654752440;

// ln x for finite x > 0; also returns the reduced mantissa's f = m - 1 and
// the exponent e
__host__ __device__ __forceinline__ double log_core(double x, double &f, int &e)
{
    double m = frexp(x, &e);  // m in [1/2, 1)
    const bool lo = m < RM_SQRT_HALF;
    m = lo ? m + m : m;
    e = lo ? e - 1 : e;
    f = m - 1.0;
    const double s = f / (m + 1.0);
    const double z = s * s;
    // t = 3 q(z)
    double t = fma(19.0 / 21.0 * z, 1.0, 1.0);
    t = fma(17.0 / 19.0 * z, t, 1.0);
    t = fma(15.0 / 17.0 * z, t, 1.0);
    t = fma(13.0 / 15.0 * z, t, 1.0);
    t = fma(11.0 / 13.0 * z, t, 1.0);
    t = fma(9.0 / 11.0 * z, t, 1.0);
    t = fma(7.0 / 9.0 * z, t, 1.0);
    t = fma(5.0 / 7.0 * z, t, 1.0);
    t = fma(3.0 / 5.0 * z, t, 1.0);
    const double d = fma(-2.0 / 3.0 * z, t, f);
    const double lnm = fma(-s, d, f);
    const double ef = (double)e;
    return fma(ef, RM_LN2_HI, fma(ef, RM_LN2_LO, lnm));
}

__host__ __device__ __forceinline__ double rt_log(double x)
{
    double f;
    int e;
    const double y = log_core(x, f, e);
    // zero, negative, infinite and NaN arguments as the library log
    return x > 0.0 && x < INFINITY ? y : (x == 0.0 ? -INFINITY : (x > 0.0 ? x : NAN));
}

// ln(1 + u) for u >= 0 (the fits' (lambda/lambda_0)^q), with the library's
// results for infinity and NaN; u < 0 is outside its domain.
// The correction c / w = c 2^-e / m takes 1/m as 1 - f + f^2, within 5% on
// the reduced range: c is below half an ulp of w, so that costs under 0.05
// ulp.
__host__ __device__ __forceinline__ double rt_log1p(double u)
{
    const double w = 1.0 + u;
    const double c = u - (w - 1.0);
    double f;
    int e;
    const double y = log_core(w, f, e);
    const double yc = fma(ldexp(c, -e), fma(f, f, 1.0 - f), y);
    return w == 1.0 ? u : (w < INFINITY ? yc : w);
}

// The angle in [0, pi] whose cosine is c and whose squared sine is s2 (the
// angle of a flux to a face normal; NaN for NaN): asin s = s + s z P(z) with
// z = s^2 <= 1/4, for s = |c| below 1/2, and above it for s = sqrt(z), z =
// (1 - |c|)/2 = s2 / (2 (1 + |c|)), where the angle of |c| is 2 asin s.  Taken
// from s2 it is accurate next to the axis, where the arccos of a rounded cosine
// is off by up to 1.5e-8.  P is the Taylor series economised to degree 12
// (truncation 6e-18 of s).  sq and rcp take the square root and the reciprocal
// (of 2 to 4), so that the device can use its own.  Within 3 ulp of pi/2 (the
// library's arccos, with its extended-precision steps, takes 95 instructions
// where this takes about 45).
template <class Sqrt, class Rcp>
__host__ __device__ __forceinline__ double angle_by(double c, double s2, Sqrt sq, Rcp rcp)
{
    const double a = fabs(c);
    const bool lo = a < 0.5;
    const double z = lo ? a * a : s2 * rcp(fma(2.0, a, 2.0));
    const double s = lo ? a : sq(z);
    double p = 0.02887841469852491;
    p = fma(p, z, -0.015032237280391934);
    p = fma(p, z, 0.01751888085821353);
    p = fma(p, z, 0.0054131676144869465);
    p = fma(p, z, 0.010333375993731042);
    p = fma(p, z, 0.011477516429392312);
    p = fma(p, z, 0.013971387140587302);
    p = fma(p, z, 0.017352380706075185);
    p = fma(p, z, 0.022372173467199163);
    p = fma(p, z, 0.030381944125004966);
    p = fma(p, z, 0.04464285714653528);
    p = fma(p, z, 0.0749999999999834);
    p = fma(p, z, 0.16666666666666669);
    const double r = fma(s, z * p, s);  // asin s
    // of |c|: pi/2 - r, or 2 r; then by the sign of c
    const double y = lo ? 1.5707963267948966 - r : r + r;
    return c < 0.0 ? 3.141592653589793 - y : y;
}

}  // namespace rtm1
