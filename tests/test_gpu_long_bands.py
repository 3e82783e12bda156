"""Bands so long that a row's byte offsets pass 2^32: every point must get its own
coefficients (transparent cells, so the intensity is the source times the path)."""
import numpy as np
import pytest

from paper_2604_11856_amd import lrt, synth

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
