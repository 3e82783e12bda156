"""Coefficients over the number of groups a workgroup's rounds of lines are shared
by: workgroups on both sides of each step of the rule, line lists that end in
the first round, at its last line and in each group of a later one, and a list
too sparse to be shared; every cell against the FP64 oracle.  The groups' sums
are added in double precision, so the tolerances are those of the terms: 1e-6
of a row's largest value in single precision (rounding of a term's centre, width
and strength, under 8 ulp), 1e-12 in double precision (exponents of some tens)."""
import numpy as np
import pytest

import torch

import oracle as O
from paper_2604_11856_amd import lrt, synth
from parity_util import edge_mask, normwise, say

pytestmark = pytest.mark.gpu
TOL = {lrt.LRT_FP32_COMP: 1e-6, lrt.LRT_FP64: 1e-12}


def _case(n_cells, n_lines, n_points, seed):
    """Lines whose windows reach over the whole grid; cells repeat three states."""
    rng = np.random.Generator(np.random.PCG64(seed))
    species = [synth.atom_species(rng, "N"), synth.atom_species(rng, "O"), synth.none_species("e-")]
    lo, steps = 40000.0, 5.0
    h = 7.16e-7 / 2.0 * np.sqrt(8000.0 / 15.0) * lo / steps
    hi = lo + h * (n_points - 1)
    nu0 = np.sort(rng.uniform(lo - 60.0 * steps * h, hi + 60.0 * steps * h, n_lines))
    z = np.zeros(n_lines)
    Eu = rng.uniform(80000.0, 110000.0, n_lines)
    lines = synth.Lines(nu0, 10 ** rng.uniform(5, 8, n_lines), Eu, z.copy(), Eu - nu0, z.copy(),
                        rng.integers(2, 13, n_lines).astype(float), rng.integers(2, 13, n_lines).astype(float),
                        rng.integers(0, 2, n_lines).astype(np.int32))
    T, N, ne = rng.uniform(5000.0, 12000.0, 3), 10 ** rng.uniform(14, 16, (3, 3)), np.array([1e15, 3e17, 1e13])

    def workload(i):
        return synth.Workload("groups", species, lines, synth.Cells(T[i], T[i] * 1.1, N[i], ne[i]),
                              synth.Grid(lo, hi, n_points, n_points), synth.SlabGeometry(np.full(i.size, 0.1), 1))

    return workload(np.arange(3)), workload(np.arange(n_cells) % 3)


# 1,100 points are three workgroups per cell: 255 and 258 workgroups, 510 and
# 513, 1,023 and 1,026
@pytest.mark.parametrize("n_cells,n_lines", [
    (1, 367), (1, 366), (1, 1300), (2, 512), (2, 513), (1, 768), (1, 769), (1, 1024), (1, 1025),
    (85, 900), (86, 900), (170, 900), (171, 900), (341, 900), (342, 900)])
@pytest.mark.parametrize("prec", [lrt.LRT_FP32_COMP, lrt.LRT_FP64])
def test_groups_against_oracle(n_cells, n_lines, prec):
    import torch
    n_points = 1100
    three, wl = _case(n_cells, n_lines, n_points, n_lines)
    say("groups: cells", n_cells, "lines", n_lines, "prec", prec)
    ref_e, ref_k, _ = O.coeffs(three.species, three.lines, three.cells, three.grid)
    m = edge_mask(three, 0, n_points)
    ctx = lrt.Context(0).load(wl)
    eta, kap, esc = ctx.coeffs_torch(0, prec)
    torch.cuda.synchronize()
    e, k = (lrt.scaled_to_f64(eta, kap, esc) if prec == lrt.LRT_FP32_COMP
            else (eta.cpu().numpy(), kap.cpu().numpy()))
    ctx.close()
    i = np.arange(n_cells) % 3
    assert normwise(e, ref_e[i], m[i]) <= TOL[prec]
    assert normwise(k, ref_k[i], m[i]) <= TOL[prec]
