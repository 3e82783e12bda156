"""The launch plan of the march (march_plan, lrt_internal.h) compiled for the host:
for any numbers of rays, cells and points its chunks cover the band once, the
kernel exists, and a caller's buffer that holds 256-point chunks is enough.
CPU only."""
import ctypes as C
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
SHIM = r'''
#include "lrt_internal.h"
extern "C" void plan(long long rays, long long cells, int band, int fp32, long long cap, long long *out)
{
    const lrt::MarchPlan p = lrt::march_plan(rays, cells, band, fp32 != 0, cap);
    out[0] = p.ppt; out[1] = p.rays; out[2] = p.n_chunks; out[3] = p.shared; out[4] = p.lds;
}
'''


@pytest.fixture(scope="module")
def shim(tmp_path_factory):
    d = tmp_path_factory.mktemp("plan")
    (d / "shim.cpp").write_text(SHIM)
    so = str(d / "shim.so")
    subprocess.run(["g++", "-std=c++17", "-O1", "-w", "-fsanitize=undefined", "-fno-sanitize-recover=all",
                    "-static-libubsan", "-shared", "-fPIC", "-D__HIP_PLATFORM_AMD__", "-I", "/opt/rocm/include",
                    "-I", os.path.join(ROOT, "paper_2604_11856_amd", "csrc"), str(d / "shim.cpp"), "-o", so], check=True)
    return C.CDLL(so)


def test_plans_hold(shim):
    rng = np.random.Generator(np.random.PCG64(4))
    edges = [1, 2, 100, 127, 128, 129, 255, 256, 257, 1279, 1280, 1281, 1792, 1793, 2 ** 30, 2 ** 31 - 256, 2 ** 31 - 1]
    out = (C.c_longlong * 5)()
    seen = set()
    for i in range(20000):
        band = edges[i % len(edges)] if i % 2 else int(2.0 ** rng.uniform(0.0, 31.0) - 1) + 1
        rays = int(rng.choice([1, 255, 256, 1024, 2048, 4095, 4096])) if i % 3 else int(2.0 ** rng.uniform(0.0, 20.0))
        cells = int(2.0 ** rng.uniform(0.0, 18.0))
        wide = rays * -(-band // 256)
        cap = [2 ** 63 - 1, wide, wide + int(rng.integers(0, wide + 1))][int(rng.integers(0, 3))]
        shim.plan(C.c_longlong(rays), C.c_longlong(cells), band, int(rng.integers(0, 2)), C.c_longlong(cap), out)
        ppt, per, chunks, shared, lds = (int(v) for v in out)
        assert ppt in (2, 4) and per in (1, 4)
        assert (chunks - 1) * 64 * ppt < band <= chunks * 64 * ppt
        assert rays * chunks <= cap
        assert lds == 0 or (shared and lds * 4 <= 160 * 1024)
        assert per == 4 or not shared
        seen.add((ppt, per, shared, lds > 0))
    # 2 and 4 points x one ray and four rays, shared, 4 of them with LDS
    assert len(seen) == 7
