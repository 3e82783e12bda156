"""Sums after the march: the spectral integral of every ray over its chunks'
partials, the flux of every wall point over its rays, and the intensities summed
over a solve's ranges, against numpy sums of the same call's outputs.  All in
double precision: the two sides add the same positive numbers in different
orders, so they agree within (terms) x 2^-53; the bar is 1e-12."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library uses)

from paper_2604_11856_amd import lrt, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_points", [1, 255, 256, 257, 700, 16 * 256, 64 * 256 + 3, 300 * 256 + 77])
@pytest.mark.parametrize("n_mu", [0, 2, 70])
def test_spectral_sums(n_points, n_mu):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(n_points)
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    grid = synth.Grid(20000.0, 20000.0 + 0.05 * n_points, n_points + 1, n_points)
    ctx.set_grid(grid)
    ctx.set_cells(synth.Cells(np.full(3, 5000.0), np.full(3, 5000.0), np.ones((3, 1)), np.ones(3)))
    ctx.set_rays(synth.SlabGeometry(np.full(3, 0.1), n_mu))
    eta = torch.rand((3, n_points), dtype=torch.float64, device="cuda:0", generator=g) + 0.1
    kap = torch.rand((3, n_points), dtype=torch.float64, device="cuda:0", generator=g)
    I = torch.empty((n_mu + 1, n_points), dtype=torch.float64, device="cuda:0")
    s = torch.empty(n_mu + 1, dtype=torch.float64, device="cuda:0")
    ctx.march(0, lrt.LRT_FP64, eta, kap, None, I, s)
    torch.cuda.synchronize()
    w = np.full(n_points, (grid.nu_max - grid.nu_min) / n_points)
    w[0] *= 0.5
    ref = I.cpu().numpy() @ w
    assert np.max(np.abs(s.cpu().numpy() - ref) / ref) <= 1e-12
    ctx.close()


@pytest.mark.parametrize("n_mu,n_phi", [(1, 1), (3, 5), (9, 14), (8, 16), (13, 10)])
@pytest.mark.parametrize("band", [700, 2000, 333])
def test_wall_and_range_sums(n_mu, n_phi, band):
    wl = synth.axisymmetric(nx=7, nr=5, n_atomic=40, n_rovib=80, n_points=2000, band_points=band, n_wall=5,
                            n_mu=n_mu, n_phi=n_phi, n_v=4, seed=n_mu)
    ctx = lrt.Context(0).load(wl)
    w = np.array([ctx.ray(r)[2:] for r in range(ctx.sizes()["n_rays"])])
    for prec in (lrt.LRT_FP64, lrt.LRT_FP32_COMP):
        for _ in range(2):   # a second solve starts its sums anew
            q, I_int, qb = ctx.solve(prec)
        ref = np.bincount(w[:, 1].astype(int), w[:, 0] * I_int)
        assert np.max(np.abs(q - ref) / ref) <= 1e-12
        assert np.max(np.abs(qb.sum(1) - q) / q) <= 1e-12
    ctx.close()
