// rt_device.h -- device-side physics of the M1 RT step for gfx950.
//
// Closure (Sec. 2, eqs. edd2/eddTens/Udir), intercell fluxes (Sec. 3.2,
// eqs. glf/hll) and the App. E rate coefficients with their T-derivatives.
// The smooth rates come from the piecewise polynomials of rt_rates.h, the
// Boltzmann factors from one sqrt(T) and 1/T per temperature.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "rt_math.h"
#include "rt_rates.h"

// Multiplies and adds are fused into FMAs only where they form one source
// expression (a * b + c): the front end marks exactly those, and the
// back end fuses every marked one, so the choice does not depend on the
// kernel that inlines a function.  A cell's result must not depend on the
// kernel that computes it (first pass or queue, grid or batch, step or
// tape); fusing across statements, as the compiler's "fast" mode may,
// could differ between kernels.  The pragma holds to the end of each
// translation unit that includes this header.
#pragma clang fp contract(on)

namespace rtm1 {

constexpr double KB = 1.380649e-16;     // erg/K
constexpr double EVERG = 1.602176634e-12;
constexpr double EPS_HI = 13.60 * EVERG;  // App. E.4 threshold table
constexpr double EPS_HEI = 24.59 * EVERG;
constexpr double EPS_HEII = 54.42 * EVERG;

// Reciprocal: the hardware v_rcp_f32 (1 ulp) in FP32 transport, IEEE
// division in FP64.
__device__ __forceinline__ float rcp(float x) { return __builtin_amdgcn_rcpf(x); }
__device__ __forceinline__ double rcp(double x) { return 1.0 / x; }

// FP64 reciprocal and quotient for a denominator b >= 1/2 (finite), as the
// rate coefficients and the helium updates have: the hardware reciprocal
// refined by two Newton steps (within an ulp), and for the quotient one
// correction from its residual.  The IEEE division's range scaling and
// special-case fix-ups are not needed there.
__device__ __forceinline__ double rcp_pos(double b)
{
    double r = __builtin_amdgcn_rcp(b);
    double e = fma(-b, r, 1.0);
    r = fma(r, e, r);
    e = fma(-b, r, 1.0);
    return fma(r, e, r);
}
__device__ __forceinline__ double div_pos(double a, double b)
{
    const double r = rcp_pos(b);
    const double q = a * r;
    const double rem = fma(-b, q, a);
    return fma(rem, r, q);
}

// The divisions, roots and angles of the transport whose arguments are
// ordinary (neither zero nor overflowing): in FP32 the hardware reciprocal and
// the library's root and arccos; in FP64 the reciprocal and the root from
// the hardware's estimates and Newton steps (5 and 9 instructions where the
// IEEE forms with their scaling and fix-ups take 11 and 18) and the angle of
// rt_math.h.
__device__ __forceinline__ float rcp_ord(float x) { return rcp(x); }
__device__ __forceinline__ double rcp_ord(double x) { return rcp_pos(x); }
__device__ __forceinline__ float sqrt_ord(float x) { return sqrt(x); }
__device__ __forceinline__ double sqrt_ord(double x)
{
    // the Goldschmidt steps of sqrt_and_inv; zero (and what underflows in the
    // square) stays zero
    const double r = __builtin_amdgcn_rsq(fmax(x, 1e-300));
    double g = x * r, h = 0.5 * r;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    return fma(fma(-g, g, x), h, g);
}
// 1/sqrt(x)
__device__ __forceinline__ float rsqrt_ord(float x) { return 1.0f / sqrt(x); }
__device__ __forceinline__ double rsqrt_ord(double x)
{
    double r = __builtin_amdgcn_rsq(x);
    double e = fma(-x * r, r, 1.0);
    r = fma(0.5 * r, e, r);
    e = fma(-x * r, r, 1.0);
    return fma(0.5 * r, e, r);
}
// the angle of cosine c, whose other two direction components are u and v
// (FP32: from the cosine alone)
__device__ __forceinline__ float angle_of(float c, float, float) { return acos(c); }
__device__ __forceinline__ double angle_of(double c, double u, double v)
{
    return angle_by(
        c, u * u + v * v, [](double z) { return sqrt_ord(z); }, [](double x) { return rcp_pos(x); });
}

// ---------------------------------------------------------------------
// M1 pressure flux.  For a cell state U = (N, F) the physical flux along
// axis d is G_d = (F_d, c^2 P_d.), P = N D with
//   D = (1-chi)/2 I + (3chi-1)/2 n (x) n,  chi = (3+4f^2)/(5+2 sqrt(4-3f^2)),
//   f = |F|/(c N) capped at 1, n = F/|F|.
// Evaluated in the scaled variable a = F/(c N) so that no square of a
// tiny density underflows (light fronts carry N down to the bottom of the
// FP32 range): with s = |a|^2 and r = sqrt(4-3s),
//   (3chi-1)/(2s) = (3/(2+r) + 6)/(5+2r)   (smooth at s = 0), hence
//   c^2 P = c^2 N [ (1-chi)/2 I + B a (x) a ],  B = (3chi-1)/(2s) for s <= 1
//   and B = 1/s (chi = 1, n = a/|a|) when the flux exceeds c N.
// Outputs the 6 independent components of c^2 P: xx, yy, zz, xy, xz, yz.
// ---------------------------------------------------------------------
template <typename R>
__device__ __forceinline__ void m1_pressure(R N, R Fx, R Fy, R Fz, R c, R P[6])
{
    const R cN = c * N;
    const R icN = rcp(cN);
    // empty cells (and densities so close to zero that 1/(c N) overflows)
    // carry no pressure
    if (!(N > R(0)) || isinf(icN)) {
#pragma unroll
        for (int k = 0; k < 6; ++k) P[k] = R(0);
        return;
    }
    const R ax = Fx * icN, ay = Fy * icN, az = Fz * icN;
    const R sr = ax * ax + ay * ay + az * az;
    const R s = sr > R(1) ? R(1) : sr;
    const R r = sqrt_ord(R(4) - R(3) * s);
    const R inv = rcp_ord(R(5) + R(2) * r);
    const R chi = (R(3) + R(4) * s) * inv;
    const R c2N = c * cN;
    const R iso = R(0.5) * (R(1) - chi) * c2N;
    const R B = (sr > R(1) ? rcp(sr) : (R(3) * rcp_ord(R(2) + r) + R(6)) * inv) * c2N;
    P[0] = iso + B * ax * ax;
    P[1] = iso + B * ay * ay;
    P[2] = iso + B * az * az;
    P[3] = B * ax * ay;
    P[4] = B * ax * az;
    P[5] = B * ay * az;
}

// After an HLL update a flux above c N is scaled back to c N: at f > 1 the
// capped closure propagates a backward wave that the table's speeds (both
// +c at f = 1) do not resolve, and an exact beam next to its source face
// would grow it from rounding.  A negative density (with speeds that
// contain each cell's reduced flux only rounding leaves one, next to a
// beam) empties the cell; vanishing densities are left.
template <typename R>
__device__ __forceinline__ void limit_flux(R &N, R &Fx, R &Fy, R &Fz, R c)
{
    if (N < R(0)) {
        N = Fx = Fy = Fz = R(0);
        return;
    }
    const R icN = rcp(c * N);
    if (!(N > R(0)) || isinf(icN)) return;
    const R ax = Fx * icN, ay = Fy * icN, az = Fz * icN;
    const R a2 = ax * ax + ay * ay + az * az;
    if (a2 > R(1)) {
        const R s = a2 < R(1e30) ? rsqrt_ord(a2) : R(1) / sqrt(a2);
        Fx *= s;
        Fy *= s;
        Fz *= s;
    }
}

// components (c^2 P_dx, c^2 P_dy, c^2 P_dz) of row d
template <typename R>
__device__ __forceinline__ void prow(const R P[6], int d, R &px, R &py, R &pz)
{
    if (d == 0) { px = P[0]; py = P[3]; pz = P[4]; }
    else if (d == 1) { px = P[3]; py = P[1]; pz = P[5]; }
    else { px = P[4]; py = P[5]; pz = P[2]; }
}

// ---------------------------------------------------------------------
// HLL wave speeds of a cell along axis d (units of c): bilinear in the
// table of (lambda_min, lambda_max) over f in [0,1] (nf nodes) and the flux
// angle theta in [0,pi] (nth nodes), theta = acos(F_d/|F|), widened to
// contain the cell's reduced flux f cos(theta).  The exact eigenvalues
// always contain it; the interpolated ones need not (at f = 1 the chord of
// cos(theta) between two nodes misses it by up to ~1e-4), and a range that
// excludes it lets the flux draw photons out of an empty cell upstream of
// a beam.
// ---------------------------------------------------------------------
// The part of the lookup shared by the three axes: the table row (f) and,
// per axis, ct_d = num_d * q (or 1 where the cell has no flux direction).
// These keep the IEEE root and divisions in FP64 too: next to f = 1 and an
// angle of pi/2 both speeds are near zero and the HLL weights magnify an ulp
// of f or of the direction a thousandfold.
template <typename R>
struct HllPrep {
    R num[3];
    R q;
    bool dir;  // false: isotropic (ct = 1)
    R f;
    int i;
    R wf;
};

template <typename R>
__device__ __forceinline__ HllPrep<R> hll_prep(int nf, R N, R Fx, R Fy, R Fz, R c)
{
    HllPrep<R> p;
    const R icN = rcp(c * N);
    const R m = fmax(fabs(Fx), fmax(fabs(Fy), fabs(Fz)));
    p.dir = m > R(0);
    if (N > R(0) && !isinf(icN)) {
        const R ax = Fx * icN, ay = Fy * icN, az = Fz * icN;
        const R an = sqrt(ax * ax + ay * ay + az * az);
        p.f = an > R(1) ? R(1) : an;
    } else {
        // empty cell: a beam if it carries any flux, isotropic otherwise
        p.f = p.dir ? R(1) : R(0);
    }
    // Direction cosines of F from F scaled by its largest component.  A flux
    // of subnormal size (FP32 fronts reach them) is first scaled by 2^64,
    // exactly, so that the reciprocal of that component cannot overflow.
    if (p.dir) {
        const R up = m < R(8.673617379884035e-19) ? R(18446744073709551616.0) : R(1);  // 2^-60, 2^64
        const R im = rcp(m * up);
        const R bx = (Fx * up) * im, by = (Fy * up) * im, bz = (Fz * up) * im;
        p.num[0] = bx;
        p.num[1] = by;
        p.num[2] = bz;
        p.q = rcp(sqrt(bx * bx + by * by + bz * bz));
    } else {
        p.num[0] = p.num[1] = p.num[2] = R(0);
        p.q = R(1);
    }
    const R uf = p.f * R(nf - 1);
    int i = (int)floor(uf);
    p.i = i > nf - 2 ? nf - 2 : (i < 0 ? 0 : i);
    p.wf = uf - R(p.i);
    return p;
}

template <typename R>
__device__ __forceinline__ void hll_axis(const R *__restrict__ tab, int nth, const HllPrep<R> &p, int d, R &lmin,
                                         R &lmax)
{
    R ct = p.dir ? p.num[d] * p.q : R(1);
    ct = ct > R(1) ? R(1) : (ct < R(-1) ? R(-1) : ct);
    const R th = angle_of(ct, p.num[d == 0 ? 1 : 0] * p.q, p.num[d == 2 ? 1 : 2] * p.q);
    const R ut = th * R(0.31830988618379067154) * R(nth - 1);
    int k = (int)floor(ut);
    k = k > nth - 2 ? nth - 2 : (k < 0 ? 0 : k);
    const R wf = p.wf, wt = ut - R(k);
    const R a00 = (R(1) - wf) * (R(1) - wt), a10 = wf * (R(1) - wt), a01 = (R(1) - wf) * wt, a11 = wf * wt;
    if constexpr (sizeof(R) == 8) {
        // the FP64 device table holds lambda_max only: lambda_min(f, theta) =
        // -lambda_max(f, pi - theta), whose nodes mirror (upload_hll_table)
        const R *t0 = tab + p.i * nth, *t1 = t0 + nth;
        const int j = nth - 2 - k;
        lmax = a00 * t0[k] + a10 * t1[k] + a01 * t0[k + 1] + a11 * t1[k + 1];
        lmin = -(a00 * t0[j + 1] + a10 * t1[j + 1] + a01 * t0[j] + a11 * t1[j]);
    } else {
        const R *t00 = tab + ((size_t)p.i * nth + k) * 2;
        const R *t01 = t00 + 2;
        const R *t10 = t00 + (size_t)nth * 2;
        const R *t11 = t10 + 2;
        lmin = a00 * t00[0] + a10 * t10[0] + a01 * t01[0] + a11 * t11[0];
        lmax = a00 * t00[1] + a10 * t10[1] + a01 * t01[1] + a11 * t11[1];
    }
    const R a = p.f * ct;
    lmin = lmin < a ? lmin : a;
    lmax = lmax > a ? lmax : a;
}

template <typename R>
__device__ __forceinline__ void hll_speeds(const R *__restrict__ tab, int nf, int nth, R N, R Fx, R Fy,
                                           R Fz, int d, R c, R &lmin, R &lmax)
{
    const HllPrep<R> p = hll_prep(nf, N, Fx, Fy, Fz, c);
    hll_axis(tab, nth, p, d, lmin, lmax);
}

// ---------------------------------------------------------------------
// App. E rate coefficients, case B (on-the-spot approximation, Sec. 3.3.2)
// or case A (without it).  vd holds value v and derivative d = dv/dT.  The
// Hui & Gnedin fits and powers of T come from the piecewise polynomials of
// rt_rates.h; the Boltzmann factors of collisional ionisation and excitation
// are computed here.
// ---------------------------------------------------------------------
struct vd {
    double v, d;
};

// sqrt(T) and 1/T from the hardware reciprocal square root r: g = T r and
// h = r/2 approach sqrt(T) and 1/(2 sqrt(T)); one Goldschmidt step on both,
// then a Newton correction of g from its residual T - g^2 and one more step
// on h, leave each within an ulp, and 1/T = (2h)^2.  (Zero or negative T
// gives NaN, and an attempt that fails: its cooling is NaN.)
__device__ __forceinline__ void sqrt_and_inv(double T, double &sq, double &inv)
{
    const double r = __builtin_amdgcn_rsq(T);
    double g = T * r, h = 0.5 * r;
    const double e = fma(-g, h, 0.5);
    g = fma(g, e, g);
    h = fma(h, e, h);
    const double d = fma(-g, g, T);
    g = fma(d, h, g);
    const double e2 = fma(-g, h, 0.5);
    h = fma(h, e2, h);
    const double h2 = h + h;
    sq = g;
    inv = h2 * h2;
}

// The smooth rates of the case in use (CA: case A) at one temperature after
// another, from the table x in global memory or (LDS) its copy l in LDS.
//
// The pointer to the global table comes out of a structure in memory; it is
// given its address space here, so that its reads are global (or, of the
// exponential's coefficients, which every lane shares, scalar) and not flat.
typedef const __attribute__((address_space(1))) double *gptr;
typedef const __attribute__((address_space(4))) double *sptr;

template <bool CA, bool LDS>
struct Rates {
    gptr x;
    const double *l;
    __device__ __forceinline__ Rates(const double *xx, const double *ll) : x((gptr)xx), l(ll) {}

    // The exponential's coefficients: scalar loads in the block that uses them
    // (the empty asm keeps them from being hoisted out of the subcycling loop,
    // where they would cost registers the loop does not have)
    __device__ __forceinline__ sptr expc() const
    {
        const uint64_t a = (uint64_t)x + RTX::X * sizeof(double);
        uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)a);
        const uint32_t hi = __builtin_amdgcn_readfirstlane((uint32_t)(a >> 32));
        asm volatile("" : "+s"(lo));
        return (sptr)((uint64_t)hi << 32 | lo);
    }

    // the coefficients of the fit at offset OX of the global table, OL of the
    // copy; a lane outside the copy reads the global one (a branch no wave of
    // an ordinary run enters).  The wait for those loads is kept inside the
    // branch: behind it every wave would wait there for all its outstanding
    // memory operations, the stores of the cells just finished among them
    template <int OX, int OL>
    __device__ __forceinline__ RateCoef fit(const RateAt &a) const
    {
        if constexpr (!LDS) return rate_coef<RT_XNI>(x + OX, a.n);
        const uint32_t n = a.n - (uint32_t)RT_LOFF;
        RateCoef c = rate_coef<RT_LNI>(l + OL, n < (uint32_t)RT_LNI ? n : 0u);
        if (__builtin_expect(n >= (uint32_t)RT_LNI, 0)) {
            c = rate_coef<RT_XNI>(x + OX, a.n);
            loaded(c);
        }
        return c;
    }
    template <int OX, int OL>
    __device__ __forceinline__ RateCoef mantissa(const RateAt &a) const
    {
        if constexpr (LDS) return rate_coef<RT_SUB>(l + OL, a.n % RT_SUB);
        else return rate_coef<RT_SUB>(x + OX, a.n % RT_SUB);
    }
    template <int OX, int OL>
    __device__ __forceinline__ double octave(const RateAt &a) const
    {
        const uint32_t o = a.n / RT_SUB;
        if constexpr (!LDS) return x[OX + o];
        const uint32_t n = o - (uint32_t)(RT_LOFF / RT_SUB);
        double v = l[OL + (n < (uint32_t)RT_LNOCT ? n : 0u)];
        if (__builtin_expect(n >= (uint32_t)RT_LNOCT, 0)) {
            v = x[OX + o];
            loaded(v);
        }
        return v;
    }

    // recombination cooling of HII, HeII (without d/dT: a power of T) and HeIII
    __device__ __forceinline__ void cooling(double T, vd &eHII, double &eHeII, vd &eHeIII, RateAt &at) const
    {
        at = rate_at(T);
        const RateAt a3 = rate_at(RT_HEIII_SCALE * T);
        RateCoef c = fit<RTX::E, RTL::E>(at), c3 = fit<RTX::E, RTL::E>(a3), cp = mantissa<RTX::P, RTL::P>(at);
        const double po = octave<RTX::PO, RTL::PO>(at);
        loaded(c, c3);
        eHII.v = rate_poly_d(c, at.z, eHII.d);
        eHII.d *= at.sc;
        eHeIII.v = (8.0 / RT_HEIII_SCALE) * rate_poly_d(c3, a3.z, eHeIII.d);
        eHeIII.d *= 8.0 * a3.sc;
        loaded(cp);
        eHeII = KB * T * (po * rate_poly(cp, at.z));
    }
    // T^-0.397 (at: as cooling() returned it for T)
    __device__ __forceinline__ double t397(const RateAt &at) const
    {
        RateCoef c = mantissa<RTX::Q, RTL::Q>(at);
        const double qo = octave<RTX::QO, RTL::QO>(at);
        loaded(c);
        return qo * rate_poly(c, at.z);
    }
    __device__ __forceinline__ vd alpha_HII(double T) const
    {
        const RateAt at = rate_at(T);
        RateCoef c = fit<RTX::A, RTL::A>(at);
        loaded(c);
        vd a;
        a.v = rate_poly_d(c, at.z, a.d);
        a.d *= at.sc;
        return a;
    }
    __device__ __forceinline__ void alpha_He(double T, double &aHeII, double &aHeIII) const
    {
        const RateAt at = rate_at(T), a3 = rate_at(RT_HEIII_SCALE * T);
        RateCoef c3 = fit<RTX::A, RTL::A>(a3), cp = mantissa<RTX::P, RTL::P>(at);
        const double po = octave<RTX::PO, RTL::PO>(at);
        loaded(c3, cp);
        aHeII = po * rate_poly(cp, at.z);
        aHeIII = 2.0 * rate_poly(c3, a3.z);
    }
    __device__ __forceinline__ double alpha_HeIII(double T) const
    {
        const RateAt a3 = rate_at(RT_HEIII_SCALE * T);
        RateCoef c = fit<RTX::A, RTL::A>(a3);
        loaded(c);
        return 2.0 * rate_poly(c, a3.z);
    }
    // alpha_A - alpha_B of HII, HeII and HeIII (the table of a case A context)
    __device__ __forceinline__ void excess(double T, double e[3]) const
    {
        const RateAt at = rate_at(T), a3 = rate_at(RT_HEIII_SCALE * T);
        RateCoef c = fit<RTX::DA, RTL::DA>(at);
        loaded(c);
        e[0] = rate_poly(c, at.z);
        c = fit<RTX::DA, RTL::DA>(a3);
        loaded(c);
        e[2] = 2.0 * rate_poly(c, a3.z);
        c = mantissa<RTX::P, RTL::P>(at);
        loaded(c);
        e[1] = octave<RTX::PO, RTL::PO>(at) * rate_poly(c, at.z);
        c = mantissa<RTX::PB, RTL::PB>(at);
        loaded(c);
        e[1] -= octave<RTX::PBO, RTL::PBO>(at) * rate_poly(c, at.z);
    }
};

// Below these temperatures exp(-Tj/T) underflows to exactly zero (its
// argument is below -745.14): 94,000 K / T for every Boltzmann factor of the
// cooling, the ionisation temperatures of HI, HeI and HeII for the rates.  A
// wave whose lanes are all below skips them; in a wave that does not, such a
// lane computes the same zero.  Nine attempts in ten of the lognormal boxes
// are in gas below 126 K: a front cell stays cold until its ionised fraction
// passes about a hundredth, which takes most of its substeps.
constexpr double T_COLD_COOL = 126.0, T_COLD_HI = 211.0, T_COLD_HEI = 382.0, T_COLD_HEII = 847.0;

// sqrt(T), 1/T, s5 = sqrt(T/1e5) and g = 1/(1+s5)
struct Tq {
    double sqT, invT, s5, g;
};
__device__ __forceinline__ Tq make_Tq(double T)
{
    Tq q;
    sqrt_and_inv(T, q.sqT, q.invT);
    q.s5 = q.sqT * 3.1622776601683795e-3;  // sqrt(1e-5)
    q.g = rcp_pos(1.0 + q.s5);
    return q;
}

// A sqrt(T) (1+sqrt(T/1e5))^-1 exp(-Tj/T)      (E.1)
__device__ __forceinline__ vd r_cen(sptr ec, const Tq &q, double A, double Tj)
{
    vd o;
    o.v = A * q.sqT * q.g * exp_neg(ec, -Tj * q.invT);
    const double dl = 0.5 - 0.5 * q.s5 * q.g + Tj * q.invT;  // dln v / dln T
    o.d = o.v * dl * q.invT;
    return o;
}

__device__ __forceinline__ vd beta_HI(sptr ec, const Tq &q) { return r_cen(ec, q, 5.85e-11, 157809.1); }
__device__ __forceinline__ vd beta_HeI(sptr ec, const Tq &q) { return r_cen(ec, q, 2.38e-11, 285335.4); }
__device__ __forceinline__ vd beta_HeII(sptr ec, const Tq &q) { return r_cen(ec, q, 5.68e-12, 631515.0); }

// Primordial cooling L of eq. (rate_cooling) and dL/dT, with the case B
// recombination cooling of the OTSA or (CA) the case A one; Tcmb and cpk are
// the temperature and the coefficient of the Compton term.
template <bool CA, bool LDS>
__device__ __forceinline__ void cooling(const Rates<CA, LDS> &r, double T, double Tcmb, double cpk, double ne, double nHI,
                                        double nHII, double nHeI, double nHeII, double nHeIII, double &L, double &dL)
{
    vd eHII, eHeIII;
    double eHeII, sqT, invT;
    RateAt at;
    r.cooling(T, eHII, eHeII, eHeIII, at);
    sqrt_and_inv(T, sqT, invT);
    const double cHI = ne * nHI, cHeI = ne * nHeI, cHeII = ne * nHeII;
    const double cHII = ne * nHII, cHeIII = ne * nHeIII;
    constexpr double eHeIIl = 1.0 - (CA ? 0.654 : 0.75);
    // bremsstrahlung and Compton
    const double th = 1.42e-27 * sqT;
    const double cp = cpk * (T - Tcmb);
    const double brn = ne * (nHII + nHeII + 4.0 * nHeIII);
    L = eHeII * cHeII + eHII.v * cHII + eHeIII.v * cHeIII + th * brn + cp * ne;
    // value * dln/dlnT of the terms without a d/dT of their own
    double dlog = eHeII * eHeIIl * cHeII + 0.5 * th * brn;
    if (!(T <= T_COLD_COOL)) {
        const sptr ec = r.expc();
        // collisional ionisation cooling (Cen form), three species
        const double s5 = sqT * 3.1622776601683795e-3;
        const double g = rcp_pos(1.0 + s5);
        const double cbase = sqT * g;          // sqrt(T)/(1+s5)
        const double gdl = -0.5 * s5 * g;      // dln g / dln T
        const double cdl = 0.5 + gdl;          // dln(cbase)/dlnT
        const double zHI = 1.27e-21 * cbase * exp_neg(ec, -157809.1 * invT), zHIl = cdl + 157809.1 * invT;
        const double zHeI = 9.38e-22 * cbase * exp_neg(ec, -285335.4 * invT), zHeIl = cdl + 285335.4 * invT;
        const double zHeII = 4.95e-22 * cbase * exp_neg(ec, -631515.0 * invT), zHeIIl = cdl + 631515.0 * invT;
        // collisional excitation
        const double psHI = 7.5e-19 * g * exp_neg(ec, -118348.0 * invT), psHIl = gdl + 118348.0 * invT;
        const double psHeII = 5.54e-17 * g * r.t397(at) * exp_neg(ec, -473638.0 * invT);
        const double psHeIIl = -0.397 + gdl + 473638.0 * invT;
        // dielectronic recombination
        const double ed2 = 0.3 * exp_neg(ec, -94000.0 * invT);
        const double om = 1.24e-13 * (invT * invT * sqT) * exp_neg(ec, -470000.0 * invT) * (1.0 + ed2);
        const double oml = -1.5 + 470000.0 * invT + div_pos(ed2 * 94000.0 * invT, 1.0 + ed2);
        L += (zHI + psHI) * cHI + zHeI * cHeI + (zHeII + psHeII + om) * cHeII;
        dlog += (zHI * zHIl + psHI * psHIl) * cHI + zHeI * zHeIl * cHeI +
                (zHeII * zHeIIl + psHeII * psHeIIl + om * oml) * cHeII;
    }
    dL = dlog * invT + eHII.d * cHII + eHeIII.d * cHeIII + cpk * ne;
}

}  // namespace rtm1
