"""The single-precision linear-j march of many rays on 256-point chunks, which takes
the series alone at points where a whole wave is thin: depths on both sides of
the line at 0.1, alone and one lane among others, negative and zero ones, point
by point against the oracle's nodes in double precision."""
import numpy as np
import pytest

import oracle as O
from paper_2604_11856_amd import lrt, synth

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [257, 512, 700])
@pytest.mark.parametrize("odd", [None, 0.5, 0.0999, 0.1001, 30.0, -0.05])
def test_thin_and_mixed_waves(n, odd):
    import torch
    n_mu, rng = 3071, np.random.Generator(np.random.PCG64(n))
    dx = np.array([1.0, 0.5, 2.0, 1.0])
    # mostly far below the line, where odd is given with single points of that depth
    kap = (10.0 ** rng.uniform(-6.0, -2.2, (4, n))).astype(np.float32)
    kap[:, ::17] = 0.0
    if odd is not None:
        kap[:, ::50] = odd
        kap[2, n // 2:] = odd   # and a stretch of whole waves
    eta = rng.uniform(0.5, 1.0, (4, n)).astype(np.float32)
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(synth.Grid(20000.0, 20000.0 + 0.05 * (n + 1), n + 2, n))
    ctx.set_cells(synth.Cells(np.full(4, 5000.0), np.full(4, 5000.0), np.ones((4, 1)), np.ones(4)))
    geom = synth.SlabGeometry(dx, n_mu)
    ctx.set_rays(geom)
    ctx.set_march(lrt.LRT_MARCH_LINEAR_J)
    e, k = (torch.from_numpy(a).to("cuda:0") for a in (eta, kap))
    esc = torch.zeros((4, 2), dtype=torch.int32, device="cuda:0")
    I = torch.empty((n_mu + 1, n), dtype=torch.float64, device="cuda:0")
    s = torch.empty(n_mu + 1, dtype=torch.float64, device="cuda:0")
    ctx.march(0, lrt.LRT_FP32_COMP, e, k, esc, I, s)
    got = I.cpu().numpy()
    ctx.close()
    rays = O.slab_rays(geom)[0]
    for r in (0, n_mu // 2, n_mu):   # along the normal, at 60 degrees, near the normal
        ref = O.march_linear(*rays[r], eta.astype(np.float64), kap.astype(np.float64))
        # thin: per segment three roundings (2e-7) of the attenuation and of each
        # of two positive sources.  From 0.1 on the 1.2e-7 of e^-t is 1.3e-6 of f and
        # 1.3e-5 of 1 - f and f - e, of which sources up to twice each other leave
        # half and the rest of the sum its share
        assert np.max(np.abs(got[r] - ref) / ref) <= (1e-6 if odd is None else 1e-5)
