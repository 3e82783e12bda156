"""Bands so long that a row's byte offsets pass 2^32: every point must get its own
coefficients (transparent cells, so the intensity is the source times the path);
and the last band of the longest grid, whose last tile and chunk end past 2^31."""
import numpy as np
import pytest

import oracle as O
from paper_2604_11856_amd import lrt, synth
from parity_util import normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("prec,n", [(lrt.LRT_FP64, (1 << 29) + 700), (lrt.LRT_FP32_COMP, (1 << 30) + 515)])
def test_march_of_a_long_band(prec, n):
    import torch
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(synth.Grid(20000.0, 20000.0 + 1e-5 * (n + 1), n + 2, n))
    ctx.set_cells(synth.Cells(np.full(1, 5000.0), np.full(1, 5000.0), np.ones((1, 1)), np.ones(1)))
    ctx.set_rays(synth.SlabGeometry(np.full(1, 0.5), 0))
    dt = torch.float64 if prec == lrt.LRT_FP64 else torch.float32
    kap = torch.zeros((1, n), dtype=dt, device="cuda:0")
    # (2^29 and 2^30 points on, where offsets wrapped, the value is another)
    eta = (torch.arange(n, device="cuda:0") % 16777213).to(dt).reshape(1, n)
    esc = torch.zeros((1, 2), dtype=torch.int32, device="cuda:0")
    I = torch.empty((1, n), dtype=torch.float64, device="cuda:0")
    s = torch.empty(1, dtype=torch.float64, device="cuda:0")
    ctx.march(0, prec, eta, kap, esc, I, s)
    torch.cuda.synchronize()
    ctx.close()
    I.mul_(2.0).sub_(eta)
    # exact in double precision; one rounding of the series' ln 2 in single
    worst = float(I.abs().max())
    assert worst <= (0.0 if prec == lrt.LRT_FP64 else 16777213 * 2.0 ** -22), worst


@pytest.mark.parametrize("prec,tol", [(lrt.LRT_FP64, 1e-12), (lrt.LRT_FP32_COMP, 1e-5)])
def test_end_of_the_longest_grid(prec, tol):
    import torch
    n, band = (1 << 31) - 1, 1000
    wl = synth.slab_equilibrium(n_cells=3, n_lines_per_species=40, n_points=200000, nu_min=99960.0, nu_max=100000.0,
                                n_mu=2, seed=7)
    wl.grid = synth.Grid(1000.0, 100000.0, n, band)
    ctx = lrt.Context(0).load(wl)
    b = n // band
    m = ctx.band_len(b)
    assert m == n % band and 512 < m < 1000
    dt = torch.float64 if prec == lrt.LRT_FP64 else torch.float32
    # room behind the last row, which nothing may write to
    buf = torch.full((2, 3 * m + 1024), -7.0, dtype=dt, device="cuda:0")
    eta, kap = (x[:3 * m].view(3, m) for x in buf)
    esc = torch.zeros((3, 2), dtype=torch.int32, device="cuda:0")
    ctx.coeffs(b, prec, eta, kap, esc)
    I = torch.empty((3, m), dtype=torch.float64, device="cuda:0")
    s = torch.empty(3, dtype=torch.float64, device="cuda:0")
    ctx.march(b, prec, eta, kap, esc, I, s)
    torch.cuda.synchronize()
    ctx.close()
    assert bool((buf[:, 3 * m:] == -7.0).all())
    ref_eta, ref_kap, _ = O.coeffs(wl.species, wl.lines, wl.cells, wl.grid, np.arange(n - m, n, dtype=np.int64))
    scale = 2.0 ** esc.cpu().numpy().astype(np.float64) if prec != lrt.LRT_FP64 else np.ones((3, 2))
    assert normwise(eta.cpu().numpy() * scale[:, :1], ref_eta) <= tol
    assert normwise(kap.cpu().numpy() * scale[:, 1:], ref_kap) <= tol
    ref = np.stack([O.march(c, d, ref_eta, ref_kap) for c, d in O.slab_rays(wl.geometry)[0]])
    assert normwise(I.cpu().numpy(), ref) <= tol
    w = O.trapezoid_weights(wl.grid, np.arange(n - m, n, dtype=np.int64))
    assert np.max(np.abs(s.cpu().numpy() - ref @ w) / (ref @ w)) <= tol
