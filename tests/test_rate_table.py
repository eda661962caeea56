"""The rate table of the chemistry kernels (piecewise polynomials of the App. E
fits) and the exponential of their Boltzmann factors, compiled from the header
the device uses: error against extended precision inside the table, at the
edges of intervals and octaves, for the HeIII fits read at the scaled
temperature, for d/dT; the exponential down to its underflow."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER_DIR = os.path.join(ROOT, "paper_1304_7126_amd", "csrc")

DRIVER = r"""
#include <vector>
#include "rt_rates.h"
using namespace rtm1;
static std::vector<double> tab[2];
// fit: 0 alpha_HII, 1 alpha_HeII, 2 alpha_HeIII, 3 HII cooling, 4 HeIII cooling, 5 T^-0.397, 6 alpha_A - alpha_B of HII
extern "C" void table_eval(int fit, int case_a, const double *T, double *v, double *d, long n)
{
    std::vector<double> &t = tab[case_a];
    if (t.empty()) {
        t.resize(case_a ? RTX::len_a : RTX::len_b);
        build_rate_table(case_a, t.data());
    }
    for (long i = 0; i < n; ++i) {
        const bool sc = fit == 2 || fit == 4;
        const RateAt a = rate_at(sc ? RT_HEIII_SCALE * T[i] : T[i]);
        double dz = 0.0;
        if (fit == 1 || fit == 5) {
            const int po = fit == 1 ? RTX::P : RTX::Q, oo = fit == 1 ? RTX::PO : RTX::QO;
            v[i] = t[oo + a.n / RT_SUB] * rate_poly(rate_coef<RT_SUB>(t.data() + po, a.n % RT_SUB), a.z);
            d[i] = 0.0;
        } else {
            const int o = fit == 3 || fit == 4 ? RTX::E : fit == 6 ? RTX::DA : RTX::A;
            v[i] = rate_poly_d(rate_coef<RT_XNI>(t.data() + o, a.n), a.z, dz);
            const double f = fit == 2 ? 2.0 : fit == 4 ? 8.0 / RT_HEIII_SCALE : 1.0;
            v[i] *= f;
            d[i] = dz * a.sc * f * (sc ? RT_HEIII_SCALE : 1.0);
        }
    }
}
extern "C" void exp_eval(const double *x, double *y, long n)
{
    for (long i = 0; i < n; ++i) y[i] = exp_neg(EXP_C, x[i]);
}
"""

L = np.longdouble
# A, power of T, TL, p, l0, q, r of A T^k lam^p / (1 + (lam/l0)^q)^r (App. E.2, E.3)
FITS = {
    False: [("2.753e-14", 0, "315614", "1.5", "2.74", "0.407", "2.242"),
            ("1.26e-14", 0, "570670", "0.75", "1", "1", "0"),
            ("5.506e-14", 0, "1263030", "1.5", "2.74", "0.407", "2.242"),
            ("3.435e-30", 1, "315614", "1.97", "2.25", "0.376", "3.72"),
            ("2.748e-29", 1, "1263030", "1.97", "2.25", "0.376", "3.72"),
            ("1", 0, "1", "0.397", "1", "1", "0")],
    True: [("1.269e-13", 0, "315614", "1.503", "0.522", "0.47", "1.923"),
           ("3e-14", 0, "570670", "0.654", "1", "1", "0"),
           ("2.538e-13", 0, "1263030", "1.503", "0.522", "0.47", "1.923"),
           ("1.778e-29", 1, "315614", "1.965", "0.541", "0.502", "2.697"),
           ("1.4224e-28", 1, "1263030", "1.965", "0.541", "0.502", "2.697"),
           ("1", 0, "1", "0.397", "1", "1", "0")],
}


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    d = tmp_path_factory.mktemp("rate_table")
    src = d / "drv.cpp"
    src.write_text(DRIVER)
    so = d / "drv.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-D__host__=", "-D__device__=",
                    "-I", HEADER_DIR, str(src), "-o", str(so)], check=True)
    return ctypes.CDLL(str(so))


def ptr(a):
    return a.ctypes.data_as(ctypes.c_void_p)


def evaluate(lib, fit, case_a, T):
    v, d = np.empty_like(T), np.empty_like(T)
    lib.table_eval(fit, int(case_a), ptr(T), ptr(v), ptr(d), ctypes.c_long(T.size))
    return v, d


def reference(fit, case_a, T):
    # the parameters as the FP64 constants the table is built from
    A, k, TL, p, l0, q, r = (L(float(c)) if isinstance(c, str) else c for c in FITS[case_a][fit])
    T = T.astype(L)
    lam = TL / T
    u = (lam / l0) ** q
    v = A * T ** k * lam ** p * (1 + u) ** -r
    return v, v * (k - p + r * q * u / (1 + u)) / T


def temperatures():
    rng = np.random.default_rng(3)
    edges = (2.0 ** np.arange(-6, 40))[:, None] * (1 + np.arange(16) / 16.0)
    edges = edges.ravel()
    return np.concatenate([10.0 ** rng.uniform(-2, 11, 100_000), edges, np.nextafter(edges, 0), np.nextafter(edges, np.inf)])


@pytest.mark.parametrize("case_a", [False, True])
@pytest.mark.parametrize("fit", range(6))
def test_table_against_extended_precision(lib, fit, case_a):
    """Bounds: two half-ulps of the last FMA and its leading coefficient, two
    more for the HeIII fits' scaled temperature and factor or a power's octave
    factor, one of slack (2^-53 each).  d/dT in units of v/T: the truncation
    |d| h^9 10/2^8 of a degree-10 term at h = 1/32 is below 1e-15, plus the
    rounding of eight products."""
    T = temperatures()
    v, d = evaluate(lib, fit, case_a, T)
    rv, rd = reference(fit, case_a, T)
    e = np.abs(v.astype(L) / rv - 1).astype(float)
    assert e.max() < 5 * 2.0 ** -53, (e.max(), T[e.argmax()])
    if fit not in (1, 5):
        ed = np.abs((d.astype(L) - rd) / (rv / T)).astype(float)
        assert ed.max() < 4e-15, (ed.max(), T[ed.argmax()])


def test_emission_difference(lib):
    # alpha_A - alpha_B as one polynomial: no cancellation of two rounded fits
    T = temperatures()
    v, _ = evaluate(lib, 6, True, T)
    ref = reference(0, True, T)[0] - reference(0, False, T)[0]
    scale = reference(0, True, T)[0]
    assert np.max(np.abs((v.astype(L) - ref) / scale).astype(float)) < 3 * 2.0 ** -53


def test_exponential(lib):
    rng = np.random.default_rng(4)
    x = np.concatenate([-rng.uniform(0, 708, 200_000), -10.0 ** rng.uniform(-20, 2.8, 100_000), [0.0, -0.0]])
    y = np.empty_like(x)
    lib.exp_eval(ptr(x), ptr(y), ctypes.c_long(x.size))
    e = np.abs(y.astype(L) / np.exp(x.astype(L)) - 1).astype(float)
    assert e.max() < 1.5 * 2.0 ** -52
    # zero where the device's cold-gas thresholds say so, and beyond
    z = np.array([-745.2, -94000.0 / 126.0, -157809.1 / 211.0, -285335.4 / 382.0, -631515.0 / 847.0, -1e6, -1e300, -np.inf])
    y = np.empty_like(z)
    lib.exp_eval(ptr(z), ptr(y), ctypes.c_long(z.size))
    assert np.all(y == 0.0)


@pytest.mark.parametrize("case_a", [False, True])
@pytest.mark.parametrize("fit", range(6))
def test_table_at_temperatures_no_gas_has(lib, fit, case_a):
    # down to 2^-126 K (the HeIII fits read at a quarter of it) and up to
    # 2^64 K a positive temperature has its own rates, within the bounds of
    # test_table_against_extended_precision
    rng = np.random.default_rng(9)
    edges = 2.0 ** np.arange(-126, 64)
    T = np.concatenate([2.0 ** rng.uniform(-126, 64, 100_000), edges, np.nextafter(edges[1:], 0)])
    v, d = evaluate(lib, fit, case_a, T)
    rv, rd = reference(fit, case_a, T)
    assert np.max(np.abs(v.astype(L) / rv - 1).astype(float)) < 5 * 2.0 ** -53
    if fit not in (1, 5):
        assert np.max(np.abs((d.astype(L) - rd) / (rv / T)).astype(float)) < 4e-15
