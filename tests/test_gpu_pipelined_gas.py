"""Pipelined chains whose moves meet none, one, two or three rows of 64 candidates (the rows of a block of at
most two are taken one by one), compared move by move with the oracle's chain."""
import pytest

import oracle
from paper_1408_3764_amd import workloads
from tests.helpers import chain_parity

pytestmark = pytest.mark.gpu


# candidates of a stencil of 27 cells: 2, 31, 63 (and the cells next to it more), 110 and 160
@pytest.mark.parametrize("n,L", [(40, 21.5), (250, 16.0), (500, 16.0), (110, 7.6), (160, 8.0)])
@pytest.mark.parametrize("max_disp", [0.2, 3.0])      # displacements inside a cell, and into another
@pytest.mark.parametrize("waves", [4, 8])
def test_few_rows(n, L, max_disp, waves):
    from paper_1408_3764_amd.box import Box
    wb = workloads.random_box(n, L, seed=3)
    p = oracle.make_params(wb.L, wb.rc, eps=wb.eps, sigma=wb.sigma, beta=wb.beta, mu=wb.mu, lambda3=wb.lambda3,
                           max_disp=max_disp, p_disp=wb.p_disp)
    b = Box(wb.pos, wb.L, wb.rc, beta=wb.beta, mu=wb.mu, lambda3=wb.lambda3, max_disp=max_disp, p_disp=wb.p_disp,
            max_n=n + 400, cell_cap=150, seed=7)
    b.set_launch(waves, -1)
    chain_parity(b, oracle, wb.pos, p, 7, 400, wb.beta, n + 400)
