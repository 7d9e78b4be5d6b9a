"""The log records of moves that an empty box rejects (a displacement or deletion with no particle): the type
and the flag, index -1, and nothing else, from every launch shape."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

SHAPES = [(4, 4), (2, 0), (4, 0), (8, 0), (16, 0), (4, -1), (8, -1), (4, -2), (4, -3), (8, -3)]


@pytest.mark.parametrize("waves,rows", SHAPES)
@pytest.mark.parametrize("mu", [-60.0, -6.0])     # nothing is ever inserted, or V e^mu = 1.3 particles
def test_empty_moves(waves, rows, mu):
    from paper_1408_3764_amd.box import Box
    b = Box(np.zeros((0, 3)), 8.0, 2.5, beta=1.0, mu=mu, max_n=400, cell_cap=64, seed=3)
    b.set_launch(waves, rows)
    _, log = b.step(120, counter0=0, log=True)
    empty = log[(log["flags"] & 1) != 0]
    assert len(empty) > (60 if mu == -60.0 else 0)
    assert (empty["type"] != 1).all() and (empty["index"] == -1).all() and (empty["accepted"] == 0).all()
    for f in ("dU_pair", "dU_tail", "x", "y", "z", "arg", "dW_pair"):
        assert (empty[f] == 0.0).all(), f
