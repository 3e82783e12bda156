"""The double-precision segment laws of the march (lrt_math.h), compiled for the
host with the reciprocal's own refinement steps, over every size of optical
depth a march can meet: zeros, subnormals, both sides of the branches, beyond
the range of the exponential, infinity.  CPU only, against extended precision."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r'''
#include "lrt_math.h"
using namespace lrt;
extern "C" {
void cell(int n, const double *t, double *em, double *f)
{ for (int i = 0; i < n; ++i) { const CellLaw w = cell_law(t[i]); em[i] = w.em; f[i] = w.f; } }
void linear(int n, const double *t, double *e, double *near, double *far)
{ for (int i = 0; i < n; ++i) { const LinearLaw w = linear_law(t[i]); e[i] = w.e; near[i] = w.near; far[i] = w.far; } }
}
'''
TINY = [5e-324, 1e-310, 5e-309, 2.0 ** -1024, 2.0 ** -1022, 1e-300, 1e-200, 1e-18]


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("shim")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-ffp-contract=off",
                    "-I", os.path.join(ROOT, "paper_2604_11856_amd", "csrc"), str(d / "shim.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def _call(f, t, n_out):
    out = [np.zeros_like(t) for _ in range(n_out)]
    f(t.size, *(a.ctypes.data_as(C.POINTER(C.c_double)) for a in (t, *out)))
    return out


def _depths():
    rng = np.random.Generator(np.random.PCG64(11))
    t = np.concatenate([TINY, 10.0 ** rng.uniform(-18, 2.8, 20000), [0.05, 0.3465, 0.3466, 1.04, 699.9]])
    return np.concatenate([t, -t])


def _weights(t):
    """f and the near and far weights in extended precision."""
    x = t.astype(np.longdouble)
    f = -np.expm1(-x) / x
    near, far = (1 - f) / x, (f - np.exp(-x)) / x
    a, b, fact = np.zeros_like(x), np.zeros_like(x), [np.longdouble(1)]
    for n in range(1, 30):
        fact.append(fact[-1] * n)
    for n in range(26, -1, -1):
        a, b = a * -x + 1 / fact[n + 2], b * -x + (n + 1) / fact[n + 2]
    thin = np.abs(x) < 1
    return f, np.where(thin, a, near), np.where(thin, b, far)


def test_cell_law(shim):
    t = _depths()
    em, f = _call(shim.cell, t, 2)
    fx = _weights(t)[0]
    # e^-t - 1 as the exponentials' own bound, the quotient one rounding more
    ok = np.abs(t) >= 2.0 ** -1022   # (below, e^-t - 1 is a subnormal of its own spacing)
    ref = np.expm1(-t.astype(np.longdouble))
    assert np.max(np.abs(em - ref)[ok] / np.abs(ref[ok])) <= 1.1e-15
    assert np.array_equal(em[~ok], -t[~ok])
    assert np.max(np.abs(f - fx) / fx) <= 1.4e-15


def test_linear_law(shim):
    t = _depths()
    e, near, far = _call(shim.linear, t, 3)
    _, nx, fx = _weights(t)
    assert np.max(np.abs(e - np.exp(-t.astype(np.longdouble))) / np.maximum(1, np.exp(-t.astype(np.longdouble)))) <= 1.4e-15
    # from t = 0.05 on 1 - f and f - e cancel to t/2: at most 40 times the 1.4e-15
    # of f and 1.1e-15 of e each
    assert np.max(np.abs(near - nx) / nx) <= 6e-14
    assert np.max(np.abs(far - fx) / fx) <= 1.1e-13


def test_attenuation_keeps_its_digits(shim):
    """e^-t of the linear-j law, however thick the segment, as close as the
    exponential is (below e^-708 a subnormal's spacing)."""
    t = np.abs(_depths())
    t = np.concatenate([t, np.linspace(1.0, 745.0, 5000)])
    e = _call(shim.linear, t, 3)[0]
    ref = np.exp(-t.astype(np.longdouble))
    assert np.max(np.abs(e - ref) / np.maximum(ref, 1e-307)) <= 4.5e-16


def test_ends(shim):
    t = np.array([0.0, -0.0, 700.0, 745.0, 1e5, 1e300, 1.7e308, np.inf])
    em, f = _call(shim.cell, t, 2)
    assert np.array_equal(em, np.expm1(-t))
    with np.errstate(invalid="ignore", divide="ignore"):
        assert np.array_equal(f, np.where(t == 0.0, 1.0, -np.expm1(-t) / t))
    e, near, far = _call(shim.linear, t, 3)
    assert np.max(np.abs(e - np.exp(-t))) <= 1e-300
    with np.errstate(invalid="ignore", divide="ignore"):
        g = 1.0 / t
        np.testing.assert_allclose(near, np.where(t == 0.0, 0.5, (1.0 - g) / t), rtol=1e-15)
        np.testing.assert_allclose(far, np.where(t == 0.0, 0.5, g / t), rtol=1e-15)
    for a in _call(shim.cell, np.array([np.nan]), 2) + _call(shim.linear, np.array([np.nan]), 3):
        assert np.isnan(a[0])
