// rt_rates.h -- the smooth App. E rate coefficients as piecewise polynomials
// in T, and the exponential of their Boltzmann factors.
//
// An attempt of the thermochemistry (App. A) evaluates Hui & Gnedin fits
// and powers of T (App. E.2, E.3) at four temperatures.  From their formula
// each costs a logarithm of T, two exponentials and a ln(1 + u): about 200
// dependent FP64 instructions, and the attempt is bound by exactly those, in
// issue where cells abound and in latency where one long chain of substeps
// is left.  The fits depend on T alone and vary slowly, so here every octave
// of T is cut into 16 intervals and each rate is a polynomial of degree 9 in
// the offset z from the interval's centre: nine FMAs (eighteen with d/dT),
// no logarithm.  The interval number and z come from the bits of T, exactly.
//
// Two fits serve for five rates: the HeIII fits are the HII fits of the
// temperature scaled by the ratio of their threshold temperatures,
//   alpha_HeIII(T) = 2 alpha_HII(s T),  eta_HeIII(T) = (8 / s) eta_HII(s T),
//   s = 315614 / 1263030,
// and a power of T = 2^e m is a factor per octave times a polynomial per
// interval of m.  For 0.5 K to 3e7 K that makes 75 KB (two FP64 tables of 448
// intervals), which the persistent chemistry kernels hold in LDS; a lane whose
// temperature is outside reads the same polynomials of the whole range from
// global memory, as the other kernels do.  The coefficients lie
// coefficient-major, so lanes whose temperatures are within two octaves of
// each other read different banks (or the same word): 4 cycles per read and
// wave.  Read from global memory as one 64-byte record per interval the
// same polynomials cost a cache lookup per lane and load, and the chemistry
// of 256^3 cells with many hot ones was no faster than with the formulas
// (4.95 against 4.84 ms per step).
//
// Measured with the persistent kernels that hold it (formulas / table): VALU
// instructions of the chemistry at 256^3 x 3, 200 sources, 1.68e9 / 1.06e9
// per launch; us per step 16^3 114 / 68, isothermal 32^3 103 / 62, 97 x 61 x
// 45 603 / 387, 64^3 754 / 517, 128^3 FP64 1,536 / 1,121, 256^3 mixed 4,799 /
// 4,129, without OTSA 150 x 141 x 133 1,372 / 948.
//
// The coefficients are built on the host in extended precision: the Taylor
// series of A T^k lam^p (1 + (lam/l0)^q)^-r about the centre (a binomial
// series, the power of a series and a product), lowered to degree 9 by
// economisation on the interval.  Against extended precision the
// values are within 3 ulp where the formula in FP64 is up to 30 ulp off,
// because the arguments of its exponentials carry the rounding of ln T.
#pragma once
#include <math.h>
#include <stdint.h>
#include <string.h>

namespace rtm1 {

// the fits; a table holds RF_AHII, RF_EHII and the powers of the case in use
// (those of HeIII are hydrogen's at RT_HEIII_SCALE times the temperature)
enum { RF_AHII, RF_AHEII, RF_EHII, RF_T397 };

// A T^k lam^p (1 + (lam/l0)^q)^-r with lam = TL/T (r = 0: a power of T)
struct RateFit {
    double A;
    int k;
    double TL, p, l0, q, r;
};

__host__ __device__ inline RateFit rate_fit(int fit, bool case_a)
{
    switch (fit) {
    case RF_AHII:  // alpha_HII
        return case_a ? RateFit{1.269e-13, 0, 315614.0, 1.503, 0.522, 0.47, 1.923}
                      : RateFit{2.753e-14, 0, 315614.0, 1.5, 2.74, 0.407, 2.242};
    case RF_AHEII:  // alpha_HeII without the dielectronic part
        return case_a ? RateFit{3e-14, 0, 570670.0, 0.654, 1.0, 1.0, 0.0}
                      : RateFit{1.26e-14, 0, 570670.0, 0.75, 1.0, 1.0, 0.0};
    case RF_EHII:  // recombination cooling of HII
        return case_a ? RateFit{1.778e-29, 1, 315614.0, 1.965, 0.541, 0.502, 2.697}
                      : RateFit{3.435e-30, 1, 315614.0, 1.97, 2.25, 0.376, 3.72};
    default:  // RF_T397: T^-0.397 of the HeII excitation cooling
        return RateFit{1.0, 0, 1.0, 0.397, 1.0, 1.0, 0.0};
    }
}

constexpr double RT_HEIII_SCALE = 315614.0 / 1263030.0;

constexpr int RT_SUB = 16;  // intervals per octave
constexpr int RT_DEG = 9;
constexpr int RT_COEF = RT_DEG + 1;
// octaves of the table in global memory, from 2^-129 K to 2^64 K, and of the part of
// it held in LDS, from 2^-3 K to 2^25 K (the HeIII fits read at a quarter of
// their temperature).  Beyond the global table the outermost intervals serve:
// above it recombination is 1e-20 of every other rate, below it lie
// temperatures smaller than a float holds.
constexpr int RT_XE0 = -129, RT_XNOCT = 193, RT_XNI = RT_XNOCT * RT_SUB;
constexpr int RT_LE0 = -3, RT_LNOCT = 28, RT_LNI = RT_LNOCT * RT_SUB;
constexpr int RT_LOFF = (RT_LE0 - RT_XE0) * RT_SUB;  // its first interval

// A table, in doubles: [coefficient][interval] of alpha_HII and of the HII
// cooling, [coefficient][interval of the mantissa] and [octave] of the powers
// alpha_HeII and T^-0.397; without OTSA also alpha_A - alpha_B of HII and the
// case B alpha_HeII.  X: the global table, L: the LDS copy, whose image lies
// behind the global table (IB, without OTSA IA), so that a workgroup's copy is
// one linear read.
constexpr int EXP_PAD = 16;
template <int NI, int NOCT, int EXP, int IMAGE_B, int IMAGE_A>
struct RateLayout {
    static constexpr int ni = NI;
    static constexpr int A = 0, E = A + RT_COEF * NI, P = E + RT_COEF * NI, Q = P + RT_COEF * RT_SUB,
                         PO = Q + RT_COEF * RT_SUB, QO = PO + NOCT, X = QO + NOCT, end_b = X + EXP;
    static constexpr int DA = end_b, PB = DA + RT_COEF * NI, PBO = PB + RT_COEF * RT_SUB, end_a = PBO + NOCT;
    // (images on 16 bytes)
    static constexpr int IB = (end_b + 1) / 2 * 2, IA = (end_a + 1) / 2 * 2;
    static constexpr int len_b = IB + IMAGE_B, len_a = IA + IMAGE_A;
};
// (X: the exponential's coefficients, in the global table only)
using RTL = RateLayout<RT_LNI, RT_LNOCT, 0, 0, 0>;
using RTX = RateLayout<RT_XNI, RT_XNOCT, EXP_PAD, RTL::len_b, RTL::len_a>;

// coefficients of the exponential (exp_neg)
constexpr int EXP_COEF = 10;
constexpr double EXP_C[EXP_COEF] = {2.5114882786996687e-08, 2.763265575933203e-07,  2.755722491836887e-06,
                                    2.480148543844738e-05,  0.00019841269909260645, 0.0013888888952356135,
                                    0.008333333333309507,   0.04166666666648794,    0.16666666666666702,
                                    0.5000000000000019};

// ------------------------------------------------------------ construction
constexpr int RT_SERIES = 14;  // degree of the Taylor series before economisation

// e[m - RT_DEG - 1][i]: the coefficient of z^i in the monic polynomial h^m
// 2^(1-m) (T_m - m/(m-2) T_m-2)(z/h), h the half width of an interval in
// units of the mantissa: its derivative is the Chebyshev polynomial T_m-1, so
// taking it off a z^m keeps the error of d/dz, which is the larger one, level
// over the interval.
struct EconomiseRows {
    long double e[RT_SERIES - RT_DEG][RT_SERIES + 1];
    EconomiseRows()
    {
        const long double h = 0.5L / RT_SUB;
        long double t[RT_SERIES + 1][RT_SERIES + 2] = {{1.0L}, {0.0L, 1.0L}};
        for (int m = 2; m <= RT_SERIES; ++m)
            for (int i = 0; i <= m; ++i)
                t[m][i] = (i > 0 ? 2.0L * t[m - 1][i - 1] : 0.0L) - (i <= m - 2 ? t[m - 2][i] : 0.0L);
        for (int m = RT_DEG + 1; m <= RT_SERIES; ++m)
            for (int i = 0; i <= m; ++i)
                e[m - RT_DEG - 1][i] = (t[m][i] - (i <= m - 2 ? (long double)m / (m - 2) * t[m - 2][i] : 0.0L)) *
                                       powl(h, m - i) * ldexpl(1.0L, 1 - m);
    }
};

// Coefficients in z of the fit about the centre of interval n.
inline void rate_series(const RateFit &f, int n, long double *out)
{
    constexpr int D = RT_SERIES;
    const long double cm = 1.0L + (2 * (n % RT_SUB) + 1) / (2.0L * RT_SUB);  // the centre's mantissa
    const long double c = ldexpl(cm, RT_XE0 + n / RT_SUB);
    const long double lam = (long double)f.TL / c;
    // (1 + w)^a, w = z / cm
    auto binom = [&](long double a, long double *s) {
        s[0] = 1.0L;
        for (int i = 1; i <= D; ++i) s[i] = s[i - 1] * (a - (i - 1)) / i;
    };
    long double pw[D + 1], y[D + 1];
    binom((long double)f.k - (long double)f.p, pw);
    y[0] = 1.0L;
    for (int i = 1; i <= D; ++i) y[i] = 0.0L;
    long double lead = (long double)f.A * powl(lam, (long double)f.p) * (f.k ? c : 1.0L);
    if (f.r != 0.0) {
        // b = (1 + u) / (1 + u0), y = b^-r: n b0 y_n = sum_i (-r i - (n - i)) b_i y_n-i
        const long double u0 = powl(lam / (long double)f.l0, (long double)f.q);
        long double b[D + 1];
        binom(-(long double)f.q, b);
        for (int i = 1; i <= D; ++i) b[i] *= u0 / (1.0L + u0);
        for (int m = 1; m <= D; ++m) {
            long double s = 0.0L;
            for (int i = 1; i <= m; ++i) s += (-(long double)f.r * i - (m - i)) * b[i] * y[m - i];
            y[m] = s / m;
        }
        lead *= powl(1.0L + u0, -(long double)f.r);
    }
    long double a[D + 1], sc = 1.0L;
    for (int m = 0; m <= D; ++m) {
        long double s = 0.0L;
        for (int i = 0; i <= m; ++i) s += pw[i] * y[m - i];
        a[m] = lead * s * sc;
        sc /= cm;
    }
    // economise: z^m less its row has a lower degree
    static const EconomiseRows er;
    for (int m = D; m > RT_DEG; --m)
        for (int i = 0; i < m; ++i) a[i] -= a[m] * er.e[m - RT_DEG - 1][i];
    for (int m = 0; m <= RT_DEG; ++m) out[m] = a[m];
}

// a power of T: the polynomials of one octave, relative to its value at the
// octave's start, and that value per octave
inline void build_power(const RateFit &f, double *poly, double *oct)
{
    for (int o = 0; o < RT_XNOCT; ++o)
        oct[o] = (double)((long double)f.A * powl((long double)f.TL / ldexpl(1.0L, RT_XE0 + o), (long double)f.p));
    RateFit u = f;
    u.A = 1.0;
    u.TL = 1.0;
    for (int n = 0; n < RT_SUB; ++n) {
        long double c[RT_COEF];
        rate_series(u, n - RT_XE0 * RT_SUB, c);  // the octave from 1 on
        for (int m = 0; m < RT_COEF; ++m) poly[m * RT_SUB + n] = (double)c[m];
    }
}

// tab: RTX::len_b doubles, or RTX::len_a with case_a
inline void build_rate_table(bool case_a, double *tab)
{
    for (int n = 0; n < RT_XNI; ++n) {
        long double a[RT_COEF], e[RT_COEF], b[RT_COEF];
        rate_series(rate_fit(RF_AHII, case_a), n, a);
        rate_series(rate_fit(RF_EHII, case_a), n, e);
        if (case_a) rate_series(rate_fit(RF_AHII, false), n, b);
        for (int m = 0; m < RT_COEF; ++m) {
            tab[RTX::A + m * RT_XNI + n] = (double)a[m];
            tab[RTX::E + m * RT_XNI + n] = (double)e[m];
            if (case_a) tab[RTX::DA + m * RT_XNI + n] = (double)(a[m] - b[m]);
        }
    }
    build_power(rate_fit(RF_AHEII, case_a), tab + RTX::P, tab + RTX::PO);
    for (int m = 0; m < EXP_PAD; ++m) tab[RTX::X + m] = m < EXP_COEF ? EXP_C[m] : 0.0;
    build_power(rate_fit(RF_T397, case_a), tab + RTX::Q, tab + RTX::QO);
    if (case_a) build_power(rate_fit(RF_AHEII, false), tab + RTX::PB, tab + RTX::PBO);
    // the image of the LDS copy
    double *l = tab + (case_a ? RTX::IA : RTX::IB);
    auto rows = [&](int src, int dst, int n, int sstride, int dstride) {
        for (int r = 0; r < n; ++r) memcpy(l + dst + r * dstride, tab + src + r * sstride, dstride * sizeof(double));
    };
    constexpr int o0 = RT_LOFF / RT_SUB;
    rows(RTX::A + RT_LOFF, RTL::A, RT_COEF, RT_XNI, RT_LNI);
    rows(RTX::E + RT_LOFF, RTL::E, RT_COEF, RT_XNI, RT_LNI);
    rows(RTX::P, RTL::P, 1, 0, 2 * RT_COEF * RT_SUB);  // P and Q
    rows(RTX::PO + o0, RTL::PO, 2, RT_XNOCT, RT_LNOCT);
    if (case_a) {
        rows(RTX::DA + RT_LOFF, RTL::DA, RT_COEF, RT_XNI, RT_LNI);
        rows(RTX::PB, RTL::PB, 1, 0, RT_COEF * RT_SUB);
        rows(RTX::PBO + o0, RTL::PBO, 1, 0, RT_LNOCT);
    }
}

// -------------------------------------------------------------- evaluation
// The interval of T (of the global table) and the offset from its centre.
// sc = 2^-exponent turns d/dz into d/dT.
struct RateAt {
    uint32_t n;
    double z, sc;
};

__host__ __device__ inline RateAt rate_at(double T)
{
    uint64_t b;
    memcpy(&b, &T, 8);
    const uint32_t hi = (uint32_t)(b >> 32);
    RateAt r;
    // an exponent below the table wraps to a large number: both ends are
    // clamped.  (A T that is not positive has an interval too, but none of its
    // rates is used: with T evolving the cooling's sqrt(T) is NaN and the
    // attempt fails; chem_init refuses an isothermal cell at T <= 0 and one
    // whose T is not finite.)
    const uint32_t u = (hi - ((uint32_t)(1023 + RT_XE0) << 20)) >> 16;
    r.n = u < (uint32_t)RT_XNI ? u : (hi < 0x3FF00000u ? 0u : (uint32_t)RT_XNI - 1u);
    const uint64_t vb = ((uint64_t)((hi & 0x000FFFFFu) | 0x3FF00000u) << 32) | (uint32_t)b;
    const uint64_t cb = (uint64_t)((hi & 0x000F0000u) | 0x3FF08000u) << 32;
    const uint64_t sb = (uint64_t)((2046u << 20) - (hi & 0x7FF00000u)) << 32;
    double v, c;
    memcpy(&v, &vb, 8);
    memcpy(&c, &cb, 8);
    memcpy(&r.sc, &sb, 8);
    r.z = v - c;
    return r;
}

// The coefficients of one interval.  loaded() marks the point where they must
// have arrived: the compiler, short of registers, would otherwise issue each
// read where its value is used and wait out its latency ten times over
// instead of once (this alone made an attempt about twice as slow).
struct RateCoef {
    double c[RT_COEF];
};
template <int STRIDE, class P>
__host__ __device__ inline RateCoef rate_coef(P t, uint32_t n)
{
    RateCoef r;
#pragma unroll
    for (int m = 0; m < RT_COEF; ++m) r.c[m] = t[m * STRIDE + n];
    return r;
}
__host__ __device__ inline void loaded(RateCoef &r)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile(""
                 : "+v"(r.c[0]), "+v"(r.c[1]), "+v"(r.c[2]), "+v"(r.c[3]), "+v"(r.c[4]), "+v"(r.c[5]), "+v"(r.c[6]),
                   "+v"(r.c[7]), "+v"(r.c[8]), "+v"(r.c[9]));
#endif
}
// (two intervals at once)
__host__ __device__ inline void loaded(double &v)
{
#if defined(__HIP_DEVICE_COMPILE__)
    asm volatile("" : "+v"(v));
#endif
}
__host__ __device__ inline void loaded(RateCoef &a, RateCoef &b)
{
#ifdef __HIP_DEVICE_COMPILE__
    asm volatile(""
                 : "+v"(a.c[0]), "+v"(a.c[1]), "+v"(a.c[2]), "+v"(a.c[3]), "+v"(a.c[4]), "+v"(a.c[5]), "+v"(a.c[6]),
                   "+v"(a.c[7]), "+v"(a.c[8]), "+v"(a.c[9]), "+v"(b.c[0]), "+v"(b.c[1]), "+v"(b.c[2]), "+v"(b.c[3]),
                   "+v"(b.c[4]), "+v"(b.c[5]), "+v"(b.c[6]), "+v"(b.c[7]), "+v"(b.c[8]), "+v"(b.c[9]));
#endif
}

__host__ __device__ inline double rate_poly(const RateCoef &r, double z)
{
    double p = r.c[RT_DEG];
#pragma unroll
    for (int m = RT_DEG - 1; m >= 0; --m) p = fma(p, z, r.c[m]);
    return p;
}

// value and d/dz
__host__ __device__ inline double rate_poly_d(const RateCoef &r, double z, double &d)
{
    double p = r.c[RT_DEG];
    d = p;
    p = fma(p, z, r.c[RT_DEG - 1]);
#pragma unroll
    for (int m = RT_DEG - 2; m >= 0; --m) {
        d = fma(d, z, p);
        p = fma(p, z, r.c[m]);
    }
    return p;
}

// exp(x) for x <= 0 (zero for NaN), the Boltzmann factors exp(-Tj/T): x = n
// ln 2 + r with |r| <= ln 2 / 2, and exp(r) from its Taylor series economised
// to degree 11 (truncation 1.6e-17; the last two coefficients are 1).
// Arguments below -2000 give zero as -2000 does; ldexp underflows by itself,
// so a general exponential's other range checks are left out.
//
// The coefficients are passed in (kept at the end of the global table):
// written as literals they are loop invariants, which the compiler holds in
// vector registers across the subcycling loop and, out of those, in scratch.
template <class P>
__host__ __device__ inline double exp_neg(P c, double x)
{
    x = fmax(x, -2000.0);
    const double n = rint(x * 1.4426950408889634);
    double r = fma(n, -0.6931471805599453, x);
    r = fma(n, -2.3190468138462996e-17, r);
    double p = c[0];
#pragma unroll
    for (int m = 1; m < EXP_COEF; ++m) p = fma(p, r, c[m]);
    p = fma(p, r, 1.0);
    p = fma(p, r, 1.0);
    return ldexp(p, (int)n);
}

}  // namespace rtm1
