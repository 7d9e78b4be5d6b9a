"""Species counts of a mixture through a checkpoint import that overflows a cell and the
rebuild with a larger capacity that its error asks for: every term that is a function of
them (tail energy, tail pressure, tail changes of moves) against the oracle."""
import numpy as np
import pytest

import oracle
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("cap", [20, 80])      # a wavefront sorts a cell, or a thread
@pytest.mark.parametrize("ns", [2, 3, 4])
def test_import_overflow_then_rebuild(ns, cap):
    from paper_1408_3764_amd import _lib
    from paper_1408_3764_amd.box import Box, make_moves
    eps, sigma = workloads.lorentz_berthelot([1.0, 1.2, 0.9, 1.1][:ns], [1.0, 0.8, 1.1, 0.9][:ns])
    wb = workloads.random_box(200, 14.0, rc=2.5, seed=9, species_counts=[40, 90, 25, 45][:ns - 1] +
                              [sum([40, 90, 25, 45][ns - 1:])], eps=eps, sigma=sigma)
    b = Box.from_workload(wb, max_n=400, cell_cap=cap)
    _, _, ck = b.export_state()
    # in the first cell nothing but a crowd of species 1, more than its places, half a diameter apart
    g = np.arange(cap + 30)
    crowd = 0.2 + 0.5 * np.stack([g % 5, g // 5 % 5, g // 25], axis=1)
    far = (wb.pos > 3.2).any(axis=1)
    pos = np.concatenate([wb.pos[far], crowd])
    sp = np.concatenate([wb.species[far], np.ones(len(g), dtype=np.int32)])
    with pytest.raises(_lib.GcmcError) as e:
        b.import_state(pos, dict(ck, n=len(pos)), species=sp)
    assert e.value.code == _lib.GCMC_ERR_CELL_OVERFLOW
    b.cell_build(cap + 40)
    p = oracle.make_params(wb.L, wb.rc, eps=eps, sigma=sigma, beta=wb.beta)
    counts = np.bincount(sp, minlength=ns)
    assert np.array_equal(np.bincount(b.particles()[1], minlength=ns), counts)
    ref, got = oracle.total_energy(pos, p, species=sp), b.total_energy()
    assert got["U_tail"] == pytest.approx(oracle.tail_energy(counts, p), rel=1e-12)
    assert abs(got["U_pair"] - ref["U_pair"]) <= 1e-10 * ref["sumabs"]
    # the tail term of the pressure: what P holds beside W / (3 V) and N / (beta V), to the rounding of P
    v, V = b.virial(), float(np.prod(wb.L))
    tail = v["P"] - v["W"] / (3.0 * V) - len(pos) / (wb.beta * V)
    assert abs(tail - oracle.tail_pressure(counts, p)) <= 8 * np.spacing(abs(v["P"]))
    # an insertion of each species: its tail change is a sum over the counts
    _, dt = b.delta_energy(make_moves([1] * ns, pos=np.full((ns, 3), 10.0), species=np.arange(ns)))
    for a in range(ns):
        assert dt[a] == pytest.approx(oracle.tail_delta(counts, a, 1, p), rel=1e-12)
