"""Energy and virial changes of caller-given moves in boxes of wide stencils, where eight wavefronts share a
move's rows: fewer rows than wavefronts and several windows of them, several groups of stencil cells, a
mixture, moves inside their cell, and both sides of the number of moves from which one wavefront takes a move.
Against the oracle's all-pairs sums within 1e-10 of the magnitude sum, the parity tests' bound."""
import numpy as np
import pytest

import oracle
from test_gpu_parity import _oracle_deltas
from test_gpu_trial_deltas import _moves
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu

#        n, edge, rc, cells, cell_cap, species
CASES = {
    "few particles, much room": (40, 9.0, 2.5, None, 200, 1),
    "6,000 candidates": (6000, 21.0, 2.5, [3, 3, 3], 0, 1),
    "6,000 candidates of three species": (6000, 23.0, 2.5, [3, 3, 3], 0, 3),
    "several groups of cells": (2000, 20.0, 5.0, [16, 16, 16], 16, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_shared_rows(name):
    from paper_1408_3764_amd.box import Box
    n, L, rc, cm, cap, ns = CASES[name]
    kw = {}
    if ns > 1:
        kw["eps"], kw["sigma"] = workloads.lorentz_berthelot([1.0, 1.2, 0.9], [1.0, 0.8, 1.1])
        kw["species_counts"] = [n // ns] * ns
    wb = workloads.random_box(n, L, rc=rc, seed=21, **kw)
    b = Box.from_workload(wb, max_n=n + 1, cell_m=cm, cell_cap=cap)
    i = b.info()
    assert i["n_stencil"] * i["cell_cap"] >= 4096
    p = oracle.make_params(wb.L, rc, eps=wb.eps, sigma=wb.sigma, beta=wb.beta)
    mv = _moves(wb, ns, 5)
    rp, rt, sa = _oracle_deltas(wb, p, mv)
    lim = 1e-10 * np.maximum(sa, 1e-300)
    gp, gt, gw = b.delta_energy(mv, virial=True)
    assert np.all(np.abs(gp - rp) <= lim) and np.allclose(gt, rt, rtol=1e-12, atol=1e-15)
    few = [b.delta_energy(mv[k:k + 1], virial=True) for k in range(5)]
    assert all(f[0][0] == gp[k] and f[2][0] == gw[k] for k, f in enumerate(few))
    # the same moves among so many that one wavefront takes each: the same to the rounding of the sums
    hp, _, hw = b.delta_energy(np.tile(mv, 7), virial=True)
    assert np.all(np.abs(hp - np.tile(rp, 7)) <= np.tile(lim, 7))
    assert np.all(np.abs(hw - np.tile(gw, 7)) <= 12.0 * np.tile(lim, 7))
