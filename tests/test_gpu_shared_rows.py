"""The march of many rays through more cells than the last-level cache holds rows
of (every XCD on one chunk), both segment schemes and precisions, thin to thick
spectra, bands of less than one chunk to several, against the oracle's march over
its own traced rays."""
import numpy as np
import pytest

import oracle as O
from paper_2604_11856_amd import lrt, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [37, 300, 1030])
@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("prec,tol", [(lrt.LRT_FP64, 1e-12), (lrt.LRT_FP32_COMP, 1e-5)])
def test_shared_chunk(n, linear, prec, tol):
    import torch
    nx, nr = (140, 120) if prec == lrt.LRT_FP32_COMP else (100, 84)
    n_cells, rng = nx * nr, np.random.Generator(np.random.PCG64(n))
    geom = synth.AxiGeometry(nx, nr, 100.0, 50.0, (np.arange(33) + 0.5) * 30.0 / 33, 16, 16)
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(synth.Grid(20000.0, 20000.0 + 0.05 * (n + 1), n + 2, n))
    ctx.set_cells(synth.Cells(np.full(n_cells, 5000.0), np.full(n_cells, 5000.0), np.ones((n_cells, 1)), np.ones(n_cells)))
    ctx.set_rays(geom)
    ctx.set_march(lrt.LRT_MARCH_LINEAR_J if linear else lrt.LRT_MARCH_CELL)
    n_rays = ctx.sizes()["n_rays"]
    assert n_rays >= 4096 and 8 * n_cells * 512 * (8 if prec == lrt.LRT_FP64 else 4) > 256 << 20
    dt = np.float64 if prec == lrt.LRT_FP64 else np.float32
    # optical depths per cell from 1e-5 to a few, varying slowly along the spectrum
    spec = np.interp(np.arange(n), np.arange(0, n + 40, 40), rng.uniform(-11.0, 0.5, n // 40 + 2))
    kap = np.exp(spec[None] + rng.uniform(-1.0, 1.0, (n_cells, 1))).astype(dt) / dt(0.7)
    eta = (kap * rng.uniform(0.2, 1.0, (n_cells, 1))).astype(dt)
    e, k = (torch.from_numpy(a).to("cuda:0") for a in (eta, kap))
    esc = torch.zeros((n_cells, 2), dtype=torch.int32, device="cuda:0")
    I = torch.empty((n_rays, n), dtype=torch.float64, device="cuda:0")
    s = torch.empty(n_rays, dtype=torch.float64, device="cuda:0")
    ctx.march(0, prec, e, k, esc, I, s)
    got = I.cpu().numpy()
    ctx.close()
    per = n_rays // 33
    march = O.march_linear if linear else O.march
    for w in (0, 7, 32):
        rays = O.axi_rays(geom, w)[0]   # (both halves of the azimuths, which are alike)
        assert len(rays) == 2 * per
        for r in (0, per // 3, per - 1):
            ref = march(*rays[r // 8 * 16 + r % 8], eta.astype(np.float64), kap.astype(np.float64))
            assert np.max(np.abs(got[w * per + r] - ref)) <= tol * ref.max()
    # every ray, and the sums over the points
    assert np.isfinite(got).all() and (got > 0.0).all()
    h = 0.05
    assert np.max(np.abs(s.cpu().numpy() - h * (got.sum(1) - 0.5 * got[:, 0]))) <= 1e-12 * h * got.sum(1).max()
