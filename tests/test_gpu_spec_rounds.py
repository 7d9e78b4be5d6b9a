"""The speculative kernel's rounds where later moves meet earlier accepted ones
most: small dense boxes whose stencils overlap everywhere (corrections), axes
covered whole, microcells with dropped stencil cells, a box that fills from
empty (prefactors far from their table, picks at every N).  Every launch shape
against the oracle move by move, and its work counters against the per-move
kernel's, which reads each move's candidates on the state it decides it on."""
import numpy as np
import pytest

import oracle
from helpers import chain_parity
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu

WORK = ("stencils", "candidates", "pair_evals", "in_cutoff")
# name: (n, L, rc, T, mu, cells per axis or None)
CASES = {
    "whole box in every stencil": (220, 7.6, 2.5, 1.3, -2.0, None),
    "five cells per axis": (700, 12.6, 2.5, 1.2, -2.5, None),
    "microcells, dropped corners": (300, 9.2, 2.5, 1.3, -2.0, [9, 9, 9]),
    "microcells, mixed axes": (300, 9.2, 2.5, 1.3, -2.0, [4, 7, 9]),
    "filling from empty": (0, 9.2, 2.5, 1.5, 3.0, None),
}


@pytest.mark.parametrize("waves", [2, 4, 8, 16])
@pytest.mark.parametrize("name", list(CASES))
def test_rounds(name, waves):
    from paper_1408_3764_amd.box import Box
    n, L, rc, T, mu, cm = CASES[name]
    wb = workloads.random_box(n, L, rc=rc, T=T, seed=40 + n, mu=mu)
    moves, max_n = 1200, n + 1201
    p = oracle.make_params(wb.L, rc, beta=wb.beta, mu=mu)
    kw = {"cell_m": None if cm is None else np.array(cm, dtype=np.int32), "cell_cap": 64, "max_n": max_n}
    b = Box.from_workload(wb, **kw)
    b.set_launch(waves, 0)
    b.total_energy()
    r = chain_parity(b, oracle, wb.pos, p, wb.seed, moves, wb.beta, max_n, name)
    assert np.array_equal(b.particles()[0], r["opos"])
    if not r["ties"]:
        ref = Box.from_workload(wb, **kw)
        ref.set_launch(4, 4)
        st, _ = ref.step(moves, counter0=0)
        assert [int(r["stats"][f]) for f in WORK] == [int(st[f]) for f in WORK]


@pytest.mark.parametrize("waves", [2, 4, 8, 16])
def test_rounds_with_overlaps(waves):
    """So hot that overlaps are accepted: an accepted move takes away or adds pair terms of 1e9 and
    more to later moves of its round, whose own sums are of order 100 and are compared as such."""
    from paper_1408_3764_amd.box import Box
    wb = workloads.random_box(120, 6.5, rc=2.5, T=1e9, seed=77, mu=0.0)
    moves, max_n = 600, 900
    p = oracle.make_params(wb.L, 2.5, beta=wb.beta, mu=0.0)
    b = Box.from_workload(wb, max_n=max_n, cell_cap=96)
    b.set_launch(waves, 0)
    b.total_energy()
    _, log = b.step(moves, counter0=0, log=True)
    _, _, olog = oracle.chain(wb.pos, moves, p, seed=wb.seed, max_n=max_n)
    big = 0
    for g, o in zip(log, olog):
        assert int(g["accepted"]) == int(o["accepted"]) and int(g["index"]) == int(o["index"])
        if int(o["flags"]) & 1:
            continue
        assert abs(g["dU_pair"] - o["dU_pair"]) <= 1e-10 * max(abs(o["dU_pair"]), o["sumabs"])
        big += abs(o["dU_pair"]) > 1e6
    assert big > 20
