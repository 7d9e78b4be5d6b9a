"""The whole-box passes over boxes whose particles fill a part of them only: the cells are dealt to the XCDs
in chunks, and a wavefront reads the counters of 64 of its cells at once.  Drops, slabs and lone particles
in few cells (fewer than there are chunks), in more (the last chunks short or empty) and in more than the
wavefronts of one launch look at once (a million).  Against the oracle's all-pairs sums, with the
tolerances of the parity tests (1e-10 of the magnitude sum for energies and virials, 1e-7 for gradients)."""
import numpy as np
import pytest

import oracle
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu

#        n, edges they fill, box edges, where, cells per axis, species
CASES = {
    "27 cells": (150, (7.0, 7.0, 7.0), (8.0, 8.0, 8.0), (0.5, 0.5, 0.5), None, 1),
    "105 cells": (300, (7.0, 12.0, 9.0), (7.6, 12.6, 18.0), (0.0, 0.3, 8.0), None, 1),
    "129 cells": (60, (6.0, 6.0, 40.0), (6.0, 6.0, 108.0), (0.0, 0.0, 60.0), [1, 3, 43], 1),
    "drop, 27,000 cells": (700, (11.0, 11.0, 11.0), (75.0, 75.0, 75.0), (33.0, 30.0, 50.0), None, 1),
    "drop of two species, 12,167 cells": (600, (12.0, 12.0, 12.0), (69.5, 69.5, 69.5), (1.0, 50.0, 20.0), None, 2),
    "slab, 4,480 cells": (900, (20.0, 20.0, 5.0), (20.0, 20.0, 175.5), (0.0, 0.0, 170.0), None, 1),
    "two drops, 1,061,208 cells": (400, (9.0, 9.0, 9.0), (255.5, 255.5, 255.5), (244.0, 120.0, 246.0), None, 1),
}


@pytest.mark.parametrize("name", list(CASES))
def test_particles_in_a_part_of_the_box(name):
    from paper_1408_3764_amd.box import Box
    n, fill, L, at, cm, ns = CASES[name]
    kw = {}
    if ns > 1:
        kw["eps"], kw["sigma"] = workloads.lorentz_berthelot([1.0, 1.2], [1.0, 0.8])
        kw["species_counts"] = [n // 2, n - n // 2]
    rc = 3.0 if ns > 1 else 2.5 if min(L) >= 6.5 else 2.0
    wb = workloads.random_box(n, np.array(fill), rc=rc, seed=11, **kw)
    pos = wb.pos + np.array(at)
    if "two drops" in name:
        pos[: n // 2] -= np.array([240.0, 110.0, 130.0])
        pos[-1] = [0.1, 255.4, 3.0]      # and a lone particle
    pos = np.mod(pos, L)
    b = Box(pos, L, rc, eps=wb.eps, sigma=wb.sigma, species=wb.species, max_n=n + 1, cell_m=cm)
    p = oracle.make_params(L, rc, eps=wb.eps, sigma=wb.sigma)
    ref = oracle.total_energy(pos, p, species=wb.species, per_particle=True)
    tol = 1e-10 * ref["sumabs"]
    assert abs(b.total_energy()["U_pair"] - ref["U_pair"]) <= tol
    got = b.total_energy(per_particle=True)
    assert abs(got["U_pair"] - ref["U_pair"]) <= tol
    assert np.allclose(got["e"], ref["e"], rtol=0, atol=1e-10 * np.abs(ref["e"]).max())
    v = oracle.virial(pos, p, species=wb.species)
    assert abs(b.virial()["W"] - v["W"]) <= 1e-10 * v["sumabs"]
    g, de, ds = oracle.gradients(pos, p, species=wb.species)
    out = b.backward()
    assert np.allclose(out["grad"], g, rtol=1e-7, atol=1e-7 * np.abs(g).max())
    assert np.allclose(out["d_eps"], de, rtol=1e-7, atol=1e-7 * np.abs(de).max())
    assert np.allclose(out["d_sigma"], ds, rtol=1e-7, atol=1e-7 * np.abs(ds).max())
