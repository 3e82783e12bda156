"""Bands that end inside a chunk of the march: every point once in the intensities
and in the trapezoid sums (whose weights are half at the grid's two ends), for
bands shorter than a chunk and from one to many chunks, first and last of a grid."""
import numpy as np
import pytest

import oracle as O
from paper_2604_11856_amd import lrt, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n_rays", [1, 3, 301])
@pytest.mark.parametrize("n", [2, 63, 127, 128, 129, 255, 256, 257, 383, 511, 513, 1000, 2047, 8193])
@pytest.mark.parametrize("prec", [lrt.LRT_FP64, lrt.LRT_FP32_COMP])
def test_every_point_once(n, n_rays, prec):
    import torch
    n_cells, rng = 3, np.random.Generator(np.random.PCG64(n))
    dt = torch.float64 if prec == lrt.LRT_FP64 else torch.float32
    # three bands: the first and the last hold an end of the grid (the last is shorter)
    grid = synth.Grid(20000.0, 20000.0 + 0.05 * (2 * n + n // 2), 2 * n + n // 2 + 1, n)
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(grid)
    ctx.set_cells(synth.Cells(np.full(n_cells, 5000.0), np.full(n_cells, 5000.0), np.ones((n_cells, 1)), np.ones(n_cells)))
    geom = synth.SlabGeometry(np.array([0.4, 0.7, 0.5]), n_rays - 1)
    ctx.set_rays(geom)
    esc = torch.zeros((n_cells, 2), dtype=torch.int32, device="cuda:0")
    rays = O.slab_rays(geom)[0]
    for band in range(3):
        m = ctx.band_len(band)
        eta = rng.uniform(0.1, 1.0, (n_cells, m)).astype(np.float64 if prec == lrt.LRT_FP64 else np.float32)
        kap = rng.uniform(0.01, 0.6, (n_cells, m)).astype(eta.dtype)
        I = torch.full((n_rays, m), float("nan"), dtype=torch.float64, device="cuda:0")
        s = torch.empty(n_rays, dtype=torch.float64, device="cuda:0")
        e, k = (torch.from_numpy(a).to("cuda:0") for a in (eta, kap))
        ctx.march(band, prec, e, k, esc, I, s)
        got, s = I.cpu().numpy(), s.cpu().numpy()
        pick = np.unique(np.linspace(0, n_rays - 1, 7).astype(int))
        ref = np.stack([O.march(*rays[r], eta.astype(np.float64), kap.astype(np.float64)) for r in pick])
        assert np.max(np.abs(got[pick] - ref) / ref) <= (1e-13 if prec == lrt.LRT_FP64 else 1e-6)
        w = O.trapezoid_weights(grid, np.arange(band * n, band * n + m))
        # a sum of positive terms in double precision
        assert np.max(np.abs(s - got @ w) / (got @ w)) <= 1e-13
    ctx.close()
