"""The march over its launch plans (chunks of 128 and 256 points, one ray or four
per workgroup, all XCDs on one chunk), segment lists around the 64 that a wave
takes at once, bands that end inside a chunk at odd offsets, and optical depths
from all thin to mixed, against the same recurrence in numpy in double precision.

Tolerances: double precision 1e-12; single precision 1e-5 of a ray's largest
intensity: a segment's attenuation and emission are rounded to 1.2e-7, and the
depths drawn here let the errors of at most some tens of segments survive."""
import numpy as np
import pytest

from paper_2604_11856_amd import lrt, synth

pytestmark = pytest.mark.gpu
TOL = {lrt.LRT_FP64: 1e-12, lrt.LRT_FP32_COMP: 1e-5}


def _reference(eta, kap, dx, mu, linear):
    """Wall intensity [rays, points]; linear-j as node segments."""
    I = np.zeros((mu.size, eta.shape[1]))
    n = dx.size
    ds = dx[None, :] / mu[:, None]

    def parts(t):
        f = np.where(t == 0.0, 1.0, -np.expm1(-t) / np.where(t == 0.0, 1.0, t))
        return f, np.exp(-t)

    if not linear:
        for c in range(n):
            t = kap[c][None, :] * ds[:, c:c + 1]
            f, e = parts(t)
            I = I * e + eta[c][None, :] * ds[:, c:c + 1] * f
        return I
    for m in range(n + 1):
        a, b = max(0, m - 1), min(m, n - 1)
        L = 0.5 * ((ds[:, m - 1] if m else 0.0) + (ds[:, m] if m < n else 0.0))[:, None]
        t = kap[a][None, :] * L
        thin = t < 0.2
        ts = np.where(thin, 1.0, t)
        f, e = parts(t)
        near = far = np.zeros_like(t)
        for k in range(14, -1, -1):
            fact = float(np.prod(np.arange(1.0, k + 3.0)))
            near, far = near * -t + 1.0 / fact, far * -t + (k + 1.0) / fact
        wn = np.where(thin, near, (1.0 - f) / ts)
        wf = np.where(thin, far, (f - e) / ts)
        I = I * e + L * (wf * eta[a][None, :] + wn * eta[b][None, :])
    return I


def _legendre_nodes(n):
    """Ascending Gauss-Legendre nodes by Newton steps."""
    x = -np.cos(np.pi * (np.arange(1, n + 1) - 0.25) / (n + 0.5))
    for _ in range(6 if n else 0):
        a, b = np.ones(n), x
        for k in range(2, n + 1):
            a, b = b, ((2 * k - 1) * x * b - (k - 1) * a) / k
        x = x - b * (x * x - 1.0) / (n * (x * b - a))
    return x


@pytest.mark.parametrize("n_cells,n_mu,n_points", [
    (1, 0, 1), (2, 0, 129), (63, 3, 257), (64, 3, 512), (65, 2, 301), (128, 0, 130), (129, 1, 1000),
    (5, 254, 70), (5, 255, 70), (66, 258, 333),         # around four rays per workgroup, a last group of 3
    (3, 11, 65536 + 3),                                  # 256-point chunks, one ray per workgroup
    (3, 300, 256 * 11 + 5),                              # 128-point chunks, four rays
    (3, 300, 8191), (3, 258, 8192 + 5),                  # up to and from 256-point chunks
    (3, 8190, 1024), (3, 8191, 1023), (3, 8191, 1024 + 1),   # and of very many rays
    (33000, 8192, 37), (33000, 8192, 1030),              # all XCDs on one chunk
])
@pytest.mark.parametrize("depth", [1e-4, 0.5])
@pytest.mark.parametrize("linear", [False, True])
@pytest.mark.parametrize("prec", [lrt.LRT_FP64, lrt.LRT_FP32_COMP])
def test_march_plans(n_cells, n_mu, n_points, depth, linear, prec):
    import torch
    if n_cells > 1000 and (linear or depth > 0.1):   # 33,000 steps of numpy
        pytest.skip("one large list is enough")
    if n_cells > 1000 and prec == lrt.LRT_FP64:
        n_cells //= 2   # the rule is in bytes
    rng = np.random.Generator(np.random.PCG64(n_cells + 7 * n_points))
    dt = np.float64 if prec == lrt.LRT_FP64 else np.float32
    dx = rng.uniform(0.5, 1.5, n_cells)
    # from far below to a few times `depth` per cell, and some of it zero
    kap = (depth * 10.0 ** rng.uniform(-4.0, 0.7, (n_cells, n_points))).astype(dt)
    kap[rng.random(kap.shape) < 0.02] = 0.0
    eta = rng.uniform(0.1, 1.0, (n_cells, n_points)).astype(dt)
    ctx = lrt.Context(0)
    ctx.set_species([synth.none_species("e-")])
    ctx.set_grid(synth.Grid(20000.0, 20000.0 + 0.05 * (n_points + 1), n_points + 2, n_points))
    ctx.set_cells(synth.Cells(np.full(n_cells, 5000.0), np.full(n_cells, 5000.0), np.ones((n_cells, 1)),
                              np.ones(n_cells)))
    ctx.set_rays(synth.SlabGeometry(dx, n_mu))
    ctx.set_march(lrt.LRT_MARCH_LINEAR_J if linear else lrt.LRT_MARCH_CELL)
    mu = np.concatenate([[1.0], 0.5 * (_legendre_nodes(n_mu) + 1.0)])
    # a base one element past an aligned address: rows start anywhere
    buf = torch.zeros((2, n_cells * n_points + 1), dtype=torch.from_numpy(eta).dtype, device="cuda:0")
    e, k = (b[1:].view(n_cells, n_points) for b in buf)
    e.copy_(torch.from_numpy(eta))
    k.copy_(torch.from_numpy(kap))
    esc = torch.zeros((n_cells, 2), dtype=torch.int32, device="cuda:0")
    I = torch.empty((n_mu + 1, n_points), dtype=torch.float64, device="cuda:0")
    s = torch.empty(n_mu + 1, dtype=torch.float64, device="cuda:0")
    ctx.march(0, prec, e, k, esc, I, s)
    torch.cuda.synchronize()
    # every ray of a small set, some of a large one, and of its points
    r = np.arange(n_mu + 1) if n_mu * n_points < 1 << 21 else np.sort(rng.choice(n_mu + 1, 24, replace=False))
    p = np.arange(n_points) if n_cells < 1000 else np.unique(np.concatenate([np.arange(0, n_points, 29), [n_points - 1]]))
    ref = _reference(eta[:, p].astype(np.float64), kap[:, p].astype(np.float64), dx, mu[r], linear)
    err = np.max(np.abs(I.cpu().numpy()[r][:, p] - ref) / ref.max(axis=1, keepdims=True))
    assert err <= TOL[prec], err
    ctx.close()
