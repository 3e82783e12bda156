"""Per-cell sums against the oracle through the coefficients in double precision:
partition functions of atoms and molecules whose level counts lie around the 64
lanes that share them, with rotational constants common to a state's levels (the
sums factor) and different ones.  And the per-cell scales of the single-precision
form, which do not depend on how many cells or species share the launch."""
import numpy as np
import pytest
import torch  # noqa: F401  (its HIP runtime is the one the library uses)

import oracle as O
from paper_2604_11856_amd import lrt, synth
from parity_util import edge_mask, normwise

pytestmark = pytest.mark.gpu


def _workload(n_lev, n_v, J_max, vary, seed, n_cells=3):
    rng = np.random.Generator(np.random.PCG64(seed))
    atom = synth.atom_species(rng, "N", n_lev)
    G = np.concatenate([1200.0 * np.arange(n) + rng.uniform(0, 50, n) for n in (n_v, 3)])
    B = np.concatenate([1.9 - 0.002 * np.arange(n_v) if vary else np.full(n_v, 1.9), [1.6, 1.6, 1.6]])
    D = np.concatenate([1e-6 * (1.0 + 0.1 * np.arange(n_v)) if vary else np.full(n_v, 6e-6), np.zeros(3)])
    mol = synth.Species("N2", synth.KIND_MOLECULE, 28.0, el_T=np.array([0.0, 59000.0]), el_g=np.array([1.0, 6.0]),
                        el_nv=np.array([n_v, 3], np.int32), el_Jmax=np.array([J_max, 40], np.int32), vib_G=G, vib_B=B,
                        vib_D=D)
    species = [atom, mol, synth.none_species("e-")]
    lo, hi = 20000.0, 20060.0
    nu0 = np.sort(rng.uniform(lo, hi, 12))
    sp = (np.arange(12) % 2).astype(np.int32)
    Eu = rng.uniform(60000.0, 90000.0, 12)
    rot = np.where(sp == 1, 500.0, 0.0)
    lines = synth.Lines(nu0, 10 ** rng.uniform(5, 8, 12), Eu, rot, Eu - nu0, rot.copy(), np.full(12, 4.0),
                        np.full(12, 2.0), sp)
    T = rng.uniform(3000.0, 12000.0, n_cells)
    cells = synth.Cells(T, T * rng.uniform(0.7, 1.3, n_cells), 10 ** rng.uniform(14, 17, (n_cells, 3)),
                        np.full(n_cells, 1e15))
    return synth.Workload("partition", species, lines, cells, synth.Grid(lo, hi, 601, 601),
                          synth.SlabGeometry(np.full(n_cells, 0.1), 0))


@pytest.mark.parametrize("n_lev", [1, 63, 64, 65, 130])
@pytest.mark.parametrize("n_v,J_max", [(1, 0), (2, 63), (50, 64), (64, 151), (65, 151), (70, 10)])
@pytest.mark.parametrize("vary", [False, True])
def test_partition_functions(n_lev, n_v, J_max, vary):
    wl = _workload(n_lev, n_v, J_max, vary, n_lev + n_v)
    ref_e, ref_k, _ = O.coeffs(wl.species, wl.lines, wl.cells, wl.grid)
    ctx = lrt.Context(0).load(wl)
    eta, kap, _ = ctx.coeffs_torch(0, lrt.LRT_FP64)
    m = edge_mask(wl, 0, 601)
    assert normwise(eta.cpu().numpy(), ref_e, m) <= 1e-12 and normwise(kap.cpu().numpy(), ref_k, m) <= 1e-12
    ctx.close()


def test_scales_by_cell_alone():
    wl = _workload(20, 8, 60, False, 3, n_cells=8200)
    wl.cells.N[:] = 10 ** np.random.Generator(np.random.PCG64(4)).uniform(-40, 17, wl.cells.N.shape)

    def scales(w):
        ctx = lrt.Context(0).load(w)
        esc = ctx.coeffs_torch(0, lrt.LRT_FP32_COMP)[2].cpu().numpy()
        ctx.close()
        return esc

    many = scales(wl)
    few = synth.Workload(wl.name, wl.species, wl.lines,
                         synth.Cells(wl.cells.T_tr[:37], wl.cells.T_v[:37], wl.cells.N[:37].copy(), wl.cells.n_e[:37]),
                         wl.grid, synth.SlabGeometry(np.full(37, 0.1), 0))
    assert np.array_equal(scales(few), many[:37]) and len(np.unique(many)) > 10
    # 70 species: the lines belong to the last two
    pad = [synth.none_species("x%d" % i) for i in range(67)]
    lines = synth.Lines(*(getattr(few.lines, f) for f in ("nu0", "A", "Eu_ev", "Eu_rot", "El_ev", "El_rot", "gu", "gl")),
                        few.lines.species + 68)
    N = np.concatenate([np.zeros((37, 67)), few.cells.N[:, 2:], few.cells.N[:, :2]], axis=1)
    wide = synth.Workload(few.name, pad + [few.species[2]] + few.species[:2], lines,
                          synth.Cells(few.cells.T_tr, few.cells.T_v, np.ascontiguousarray(N), few.cells.n_e),
                          few.grid, few.geometry)
    assert np.array_equal(scales(wide), many[:37])
