"""The double-precision march over optical depths of every size, zero, subnormal
and infinite ones among them, and a whole solve whose far line wings are
subnormal: finite everywhere and equal to the oracle's."""
import numpy as np
import pytest

import oracle as O
from paper_2604_11856_amd import lrt, synth
from parity_util import normwise

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("linear", [False, True])
def test_depths_of_every_size(linear):
    import torch
    t = np.array([0.0, 5e-324, 1e-310, 5e-309, 2.0 ** -1024, 2.0 ** -1022, 1e-300, 1e-200, 1e-18, 1e-9, 0.04, 0.05,
                  0.34, 0.35, 1.0, 40.0, 699.0, 701.0, 745.0, 1e5, 1e300, np.inf])
    # every depth before and after every other, the linear-j nodes half a cell off
    kap = np.concatenate([np.tile(t, t.size)[None], np.repeat(t, t.size)[None], np.tile(t, t.size)[None]])
    eta = np.broadcast_to(np.array([1.0, 0.25, 2.0])[:, None], kap.shape).copy()
    n = kap.shape[1]
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(synth.Grid(20000.0, 20000.0 + 0.05 * (n + 1), n + 2, n))
    ctx.set_cells(synth.Cells(np.full(3, 5000.0), np.full(3, 5000.0), np.ones((3, 1)), np.ones(3)))
    geom = synth.SlabGeometry(np.ones(3), 2)
    ctx.set_rays(geom)
    ctx.set_march(lrt.LRT_MARCH_LINEAR_J if linear else lrt.LRT_MARCH_CELL)
    e, k = (torch.from_numpy(a).to("cuda:0") for a in (eta, kap))
    I = torch.empty((3, n), dtype=torch.float64, device="cuda:0")
    s = torch.empty(3, dtype=torch.float64, device="cuda:0")
    ctx.march(0, lrt.LRT_FP64, e, k, None, I, s)
    got = I.cpu().numpy()
    ctx.close()
    assert np.isfinite(got).all() and np.isfinite(s.cpu().numpy()).all()
    march = O.march_linear if linear else O.march
    ref = np.stack([march(c, d, eta, kap) for c, d in O.slab_rays(geom)[0]])
    assert np.isfinite(ref).all()
    # three or four segments of positive terms, each within some roundings; the
    # linear-j weights cancel to 1.1e-13 of themselves at a depth of 0.05
    # (zero behind an infinite depth)
    assert np.max(np.abs(got - ref) / np.where(ref > 0.0, ref, 5e-324)) <= (4e-13 if linear else 1e-14)


@pytest.mark.parametrize("T", [(8000.0, 500.0, 600.0, 1000.0, 5000.0, 11000.0), (300.0, 225.0, 212.0, 8000.0)])
def test_subnormal_wings_stay_finite(T):
    wl = synth.slab_equilibrium(n_cells=len(T), dx=0.1, n_lines_per_species=500, n_points=40001, n_mu=2, seed=1)
    # without electrons the profiles are Gaussians, which end in subnormals
    wl.cells.n_e[:] = 0.0
    wl.cells.T_tr[:] = wl.cells.T_v[:] = T
    ref = O.solve_slab(wl)
    depth = ref["kappa"] * 0.1
    assert np.any((depth > 0.0) & (depth < 2.0 ** -1024))
    ctx = lrt.Context(0).load(wl)
    q, I_int, _ = ctx.solve(lrt.LRT_FP64)
    ctx.close()
    assert np.isfinite(q).all() and np.isfinite(I_int).all()
    if min(T) >= 500.0:   # (the oracle's e^x - 1 of the coldest cells overflows)
        assert normwise(I_int[None], ref["I_int"][None]) <= 1e-12
        assert abs(q[0] - ref["q"]) <= 1e-12 * ref["q"]
