"""Where the double-precision accumulation leaves the Gaussian of the profile out
(gauss_reach_f64, lrt_nodes.h): below 2^-56 of the rational part, or zero, for
every Lorentz fraction down to zero.  CPU only."""
import ctypes as C
import os
import subprocess

import numpy as np

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r'''
#include "lrt_nodes.h"
extern "C" float reach(double r) { return lrt::gauss_reach_f64(r); }
'''


def test_nothing_left_out(tmp_path):
    (tmp_path / "shim.cpp").write_text(SHIM)
    so = str(tmp_path / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O2", "-shared", "-fPIC", "-I",
                    os.path.join(ROOT, "paper_2604_11856_amd", "csrc"), str(tmp_path / "shim.cpp"), "-o", so], check=True)
    f = C.CDLL(so).reach
    f.restype, f.argtypes = C.c_float, [C.c_double]
    F = np.longdouble
    for r in [0.0, 5e-324, 2.0 ** -1050, 2.0 ** -1022, 2.0 ** -1015, 2.0 ** -1000, 2.0 ** -500, 1e-30, 1e-3, 0.5, 1.0]:
        y = F(f(r)) * np.linspace(1.0, 3.0, 400).astype(F)
        gauss = (1 - F(r)) * np.exp(F(-2.772) * (y / 2) ** 2)
        left = gauss.astype(np.float64) > 0.0
        rational = F(r) / (1 + y * y) - F(0.016) * F(r) * (1 - F(r)) / (1 + F(0.1) * (y / 2) ** F(2.25))
        assert np.all(gauss[left] <= rational[left] * F(2.0) ** -56), r
