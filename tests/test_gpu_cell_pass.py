"""The whole-box passes over the cell list (total energy, per-particle energies,
pair virial, gradient) where their work split can go wrong: boxes of 0, 1 and 2
particles, empty cells, axes covered whole, cells that are each other's
half-way partner, partly covered boxes, more than 64 particles in a cell, more
than 2,048 candidates in a stencil, more than 64 stencil cells, several species
with a non-interacting pair, overlapping particles.  Against the oracle's
all-pairs sums, with the tolerances of the parity tests (1e-10 of the magnitude
sum for energies and virials, 1e-7 for gradients)."""
import itertools

import numpy as np
import pytest

import oracle
from paper_1408_3764_amd import workloads

# name: (n, box edges, rc, cells per axis or None, species)
CASES = {
    "one": (1, 8.0, 2.5, None, 1),
    "two": (2, 8.0, 2.5, None, 1),
    "whole axes, M=3": (300, 8.0, 2.5, None, 1),
    "whole axes, M=4 even": (300, 9.0, 3.0, [4, 4, 4], 1),
    "partly whole 3x8x5": (500, (7.6, 20.2, 12.6), 2.5, None, 1),
    "empty cells": (60, 30.0, 2.5, None, 1),
    "92 per cell, 2,500 candidates": (2500, 15.4, 5.0, None, 1),
    "66 per cell, pruned edges": (1500, (13.0, 13.0, 13.0), 4.3, None, 1),
    "125 stencil cells": (900, 13.0, 2.5, [10, 10, 10], 1),
    "343 block, M=7 whole": (400, 9.0, 3.0, [7, 7, 7], 1),
    "two species": (500, 12.5, 3.0, None, 2),
    "four species": (600, 12.5, 3.0, None, 4),
    "two species, microcells": (400, 12.5, 3.0, [9, 8, 7], 2),
}


def _case(name):
    n, L, rc, cm, ns = CASES[name]
    if ns == 1:
        wb = workloads.random_box(n, L, rc=rc, seed=5 + n)
    else:
        eps, sig = workloads.lorentz_berthelot([1.0, 1.2, 0.9, 1.1][:ns], [1.0, 0.8, 1.1, 0.7][:ns])
        eps[0, ns - 1] = eps[ns - 1, 0] = 0.0     # a pair of species that does not interact
        counts = [n // ns] * (ns - 1) + [n - n // ns * (ns - 1)]
        wb = workloads.random_box(n, L, rc=rc, seed=5 + n, species_counts=counts, eps=eps, sigma=sig)
    return wb, cm, oracle.make_params(wb.L, wb.rc, eps=wb.eps, sigma=wb.sigma, beta=wb.beta)


def _box(wb, cm):
    from paper_1408_3764_amd.box import Box
    return Box.from_workload(wb, max_n=wb.n + 1, cell_m=None if cm is None else np.array(cm, dtype=np.int32))


@pytest.mark.gpu
@pytest.mark.parametrize("name", list(CASES))
def test_passes_at_edges(name):
    wb, cm, p = _case(name)
    b = _box(wb, cm)
    ref = oracle.total_energy(wb.pos, p, species=wb.species, per_particle=True)
    tol = 1e-10 * max(ref["sumabs"], 1e-300)
    assert abs(b.total_energy()["U_pair"] - ref["U_pair"]) <= tol
    got = b.total_energy(per_particle=True)
    assert abs(got["U_pair"] - ref["U_pair"]) <= tol
    assert np.allclose(got["e"], ref["e"], rtol=0, atol=1e-10 * max(1.0, np.abs(ref["e"]).max()))
    v = oracle.virial(wb.pos, p, species=wb.species)
    assert abs(b.virial()["W"] - v["W"]) <= 1e-10 * max(v["sumabs"], 1e-300)
    g, de, ds = oracle.gradients(wb.pos, p, species=wb.species)
    out = b.backward()
    assert np.allclose(out["grad"], g, rtol=1e-7, atol=1e-7 * max(np.abs(g).max(), 1e-300))
    assert np.allclose(out["d_eps"], de, rtol=1e-7, atol=1e-7 * max(np.abs(de).max(), 1e-300))
    assert np.allclose(out["d_sigma"], ds, rtol=1e-7, atol=1e-7 * max(np.abs(ds).max(), 1e-300))
    only = b.backward(params=False)["grad"]
    assert np.array_equal(only, out["grad"])


@pytest.mark.gpu
def test_passes_overlap_and_empty():
    """Overlapping particles: +inf where they interact, nothing where their epsilon is 0; an empty box: 0."""
    wb, cm, p = _case("two species")
    i, j = int(np.nonzero(wb.species == 0)[0][0]), int(np.nonzero(wb.species == 1)[0][0])
    wb.pos[j] = wb.pos[i]                      # eps_01 = 0: no interaction
    ref = oracle.total_energy(wb.pos, p, species=wb.species)
    assert abs(_box(wb, cm).total_energy()["U_pair"] - ref["U_pair"]) <= 1e-10 * ref["sumabs"]
    wb, cm, p = _case("whole axes, M=3")
    wb.pos[7] = wb.pos[200]
    b = _box(wb, cm)
    assert np.isposinf(b.total_energy()["U_pair"]) and np.isposinf(b.virial()["W"])
    e = b.total_energy(per_particle=True)["e"]
    assert np.array_equal(np.nonzero(np.isinf(e))[0], [7, 200])
    assert np.isfinite(b.backward()["grad"]).all()
    from paper_1408_3764_amd.box import Box
    empty = Box(np.zeros((0, 3)), 10.0, 2.5, max_n=4)
    assert empty.total_energy()["U_pair"] == 0.0 and empty.virial()["W"] == 0.0


@pytest.mark.parametrize("M,k", [((3, 3, 3), (1, 1, 1)), ((4, 4, 4), (1, 2, 2)), ((3, 8, 5), (1, 1, 2)),
                                 ((5, 4, 2), (1, 1, 1)), ((7, 7, 7), (3, 3, 3)), ((6, 5, 4), (2, 1, 1))])
def test_each_pair_of_cells_from_one_side(M, k):
    """The rule that lets a home cell c take a stencil cell c' (2 d < cells, d = c' - c modulo
    the number of cells; c < c' at equality) takes every pair of cells of a symmetric stencil once."""
    cells = M[0] * M[1] * M[2]
    full = [2 * k[a] + 1 >= M[a] for a in range(3)]
    taken = {}
    for c in range(cells):
        at = (c % M[0], c // M[0] % M[1], c // (M[0] * M[1]))
        axes = [range(M[a]) if full[a] else [(at[a] + o) % M[a] for o in range(-k[a], k[a] + 1)] for a in range(3)]
        for x, y, z in itertools.product(*axes):
            o = (z * M[1] + y) * M[0] + x
            if o != c:
                d2 = 2 * ((o - c) % cells)
                taken.setdefault(frozenset((c, o)), []).append(d2 < cells or (d2 == cells and c < o))
    assert all(len(v) == 2 and sum(v) == 1 for v in taken.values())
