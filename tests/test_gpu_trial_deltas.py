"""Energy and virial changes of caller-given moves where the stencil pass can go
wrong: displacements inside a cell (both positions share the candidates), across
cells and through the periodic wall, insertions into empty stencils and onto a
particle, refused indices and species among accepted moves, whole axes, stencils
of 125 cells, more candidates than one window of rows, several species.  Against
the oracle's all-pairs sums within 1e-10 of the magnitude sum, the parity tests'
bound, and against the all-pairs kernel for the virial change (the sum of two
independent orders: twice that bound, the virial's own magnitudes from the
oracle's pair sums being at most 12 times the energy's)."""
import numpy as np
import pytest

import oracle
from test_gpu_cell_pass import _box, _case
from test_gpu_parity import _oracle_deltas


def _moves(wb, ns, seed):
    from paper_1408_3764_amd.box import make_moves
    rng = np.random.default_rng(seed)
    n, L = wb.n, np.asarray(wb.L)
    m = 160
    types = rng.integers(0, 3, m)
    idx = rng.integers(0, n, m)
    step = np.where(rng.random((m, 1)) < 0.5, 0.05, 0.4 * L)      # mostly the same cell, or anywhere
    p = np.where((types == 0)[:, None], wb.pos[idx] + rng.uniform(-1, 1, (m, 3)) * step, rng.random((m, 3)) * L)
    p = np.mod(p, L)
    p[p >= L] = 0.0
    mv = make_moves(types, idx, p)
    mv["species"] = rng.integers(0, ns, m)
    return mv


@pytest.mark.gpu
@pytest.mark.parametrize("name", ["one", "two", "whole axes, M=3", "partly whole 3x8x5", "empty cells",
                                  "92 per cell, 2,500 candidates", "125 stencil cells", "343 block, M=7 whole",
                                  "two species", "four species", "two species, microcells"])
def test_trials_at_edges(name):
    wb, cm, p = _case(name)
    ns = 1 if wb.species is None else wb.eps.shape[0]
    b = _box(wb, cm)
    mv = _moves(wb, ns, 11)
    rp, rt, sa = _oracle_deltas(wb, p, mv)
    gp, gt, gw = b.delta_energy(mv, virial=True)
    assert np.all(np.abs(gp - rp) <= 1e-10 * np.maximum(sa, 1e-300))
    assert np.allclose(gt, rt, rtol=1e-12, atol=1e-15)
    ap, at, aw = b.delta_energy(mv, all_pairs=True, virial=True)
    assert np.all(np.abs(gw - aw) <= 2e-10 * 12.0 * np.maximum(sa, 1e-300))
    # refused moves among accepted ones give NaN and leave their neighbours alone
    bad = mv.copy()
    bad["type"][::3], bad["index"][::3] = 2, np.where(np.arange(len(bad[::3])) % 2, wb.n, -1)
    bad["type"][1::3], bad["species"][1::3] = 1, ns
    hp, ht, hw = b.delta_energy(bad, virial=True)
    assert np.isnan(hp[::3]).all() and np.isnan(ht[1::3]).all() and np.isnan(hw[1::3]).all()
    assert np.array_equal(hp[2::3], gp[2::3]) and np.array_equal(hw[2::3], gw[2::3])
    # the order of the calls and of the moves does not enter a result
    rev, _, revw = b.delta_energy(mv[::-1], virial=True)
    assert np.array_equal(rev[::-1], gp) and np.array_equal(revw[::-1], gw)


@pytest.mark.gpu
def test_trials_on_a_particle():
    """Two coincident pairs: an insertion there is +inf, leaving is -inf, moving from one to the other NaN."""
    from paper_1408_3764_amd.box import Box, make_moves
    pos = np.array([[1.0, 1.0, 1.0], [1.0, 1.0, 1.0], [5.0, 5.0, 5.0], [7.0, 2.0, 3.0]])
    b = Box(pos, [8.0] * 3, 2.5, max_n=8)
    mv = make_moves([1, 0, 0, 2], [0, 3, 0, 0], [[5.0] * 3, [5.0] * 3, [5.0] * 3, [0.0] * 3])
    for all_pairs in (False, True):
        gp, _ = b.delta_energy(mv, all_pairs=all_pairs)
        assert gp[0] == np.inf and gp[1] == np.inf and np.isnan(gp[2]) and gp[3] == -np.inf
