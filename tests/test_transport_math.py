"""The angle of a flux to a face normal in the FP64 transport, from its cosine
and squared sine, compiled from the header the device uses, against extended
precision."""
import ctypes
import os
import shutil
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
HEADER_DIR = os.path.join(ROOT, "paper_1304_7126_amd", "csrc")

DRIVER = r"""
#include "rt_math.h"
extern "C" void ac_eval(const double *c, const double *s2, double *y, long n)
{
    for (long i = 0; i < n; ++i)
        y[i] = rtm1::angle_by(c[i], s2[i], [](double z) { return sqrt(z); }, [](double v) { return 1.0 / v; });
}
"""


def test_angle(tmp_path):
    cxx = shutil.which("g++")
    if cxx is None:
        pytest.skip("no host C++ compiler")
    src = tmp_path / "drv.cpp"
    src.write_text(DRIVER)
    so = tmp_path / "drv.so"
    subprocess.run([cxx, "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-D__host__=", "-D__device__=",
                    "-D__forceinline__=inline", "-I", HEADER_DIR, str(src), "-o", str(so)], check=True)
    lib = ctypes.CDLL(str(so))
    rng = np.random.default_rng(2)
    th = np.concatenate([rng.uniform(0, np.pi, 300_000), 10.0 ** rng.uniform(-150, 0, 50_000),
                         np.pi - 10.0 ** rng.uniform(-15, 0, 50_000), [0.0, np.pi / 3, np.pi / 2]]).astype(np.longdouble)
    c = np.cos(th).astype(float)
    s2 = (np.sin(th) ** 2).astype(float)
    y = np.empty_like(c)
    p = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    lib.ac_eval(p(c), p(s2), p(y), ctypes.c_long(c.size))
    # the rounding of c and s2, of asin s, its doubling or the difference from
    # pi/2, the difference from pi and the constants: six half-ulps of pi/2
    e = np.abs(y.astype(np.longdouble) - th).astype(float)
    assert e.max() < 3.0 * 2.0 ** -52, (e.max(), float(th[e.argmax()]))
    # small angles relative to themselves: s2, the reciprocal, the root, asin
    small = (th < 0.5) & (th > 0)
    assert np.max(e[small] / th[small].astype(float)) < 6 * 2.0 ** -53
    assert y[th == 0.0][0] == 0.0
    z = np.array([np.nan])
    lib.ac_eval(p(z), p(z), p(z), ctypes.c_long(1))
    assert np.isnan(z[0])
