"""The whole-box passes over a vapour (a lane per particle): more particles than a batch lists, cells with more
particles than are listed at once, an axis covered whole, mixtures with a non-interacting pair, the last group
of cells short, both sides of the rule that chooses them.  Totals against plain numpy sums over the pairs
that a k-d tree finds, single particles against the oracle, with the tolerances of the parity tests (1e-10 of
the magnitude sum for energies and virials, 1e-7 for gradients)."""
import numpy as np
import pytest
from scipy.spatial import cKDTree

import oracle
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu

#        n, edges, rc, cells, species, a cell of that many more
CASES = {
    "one species": (70001, (130.0, 131.0, 137.0), 2.5, None, 1, 0),
    "13 in a cell": (66000, (132.0, 132.0, 132.0), 2.5, None, 1, 13),
    "30 in a cell: a wavefront per cell": (66000, (132.0, 132.0, 132.0), 2.5, None, 1, 30),
    "an axis of three cells": (65536, (8.0, 400.0, 450.0), 2.5, None, 1, 0),
    "microcells": (80000, (110.0, 110.0, 110.0), 3.0, [72, 73, 74], 1, 0),
    "two species": (66001, (125.0, 150.0, 110.0), 2.5, None, 2, 0),
    "four species": (66001, (125.0, 150.0, 110.0), 2.5, None, 4, 0),
    "1.5 in a cell": (530000, (177.0, 177.0, 177.0), 2.5, None, 1, 0),
}


def _gas(n, L, crowd, rng):
    """Sites of a lattice 1.2 apart, jittered by 0.15, and a crowd half a diameter apart in the first cell."""
    L = np.asarray(L)
    m = np.floor(L / 1.2).astype(np.int64)
    site = rng.permutation(int(np.prod(m)))[: n - crowd]
    pos = np.stack([site % m[0], site // m[0] % m[1], site // (m[0] * m[1])], axis=1) * 1.2 + 0.6
    pos = np.mod(pos + rng.uniform(-0.15, 0.15, pos.shape), L)
    if crowd:
        pos = pos[~(pos < 3.3).all(axis=1)]
        g = np.arange(crowd + n - crowd - len(pos)) if crowd >= 13 else np.arange(n - len(pos))
        pos = np.concatenate([pos, 0.2 + 0.45 * np.stack([g % 5, g // 5 % 5, g // 25], axis=1)])
    return pos


def _sums(pos, L, rc, eps, sig, sp):
    """U_pair, W, e_i, gradient, d_eps, d_sigma (pair parts) and the magnitude sums of U and W."""
    L, ns = np.asarray(L), len(eps)
    pairs = cKDTree(pos, boxsize=L).query_pairs(rc * (1 + 1e-9), output_type="ndarray")
    i, j = pairs[:, 0], pairs[:, 1]
    d = pos[j] - pos[i]
    d -= L * np.round(d / L)
    r2 = (d * d).sum(axis=1)
    k = r2 < rc * rc
    i, j, d, r2 = i[k], j[k], d[k], r2[k]
    a, b = sp[i], sp[j]
    e, s6 = eps[a, b], (sig[a, b] ** 2 / r2) ** 3
    u, w = 4 * e * (s6 * s6 - s6), 24 * e * (2 * s6 * s6 - s6)
    each = np.bincount(i, u, len(pos)) + np.bincount(j, u, len(pos))
    g = np.zeros_like(pos)
    for x in range(3):
        f = w / r2 * d[:, x]       # dU/dr_i = -(dU/dr) d / r, d from i to j
        g[:, x] = np.bincount(i, f, len(pos)) - np.bincount(j, f, len(pos))
    de, ds = np.zeros((ns, ns)), np.zeros((ns, ns))
    for x, y in ((a, b), (b, a)):
        np.add.at(de, (x, y), 2 * (s6 * s6 - s6))
        np.add.at(ds, (x, y), 12 * e / sig[a, b] * (2 * s6 * s6 - s6))
    return u.sum(), w.sum(), each, g, de, ds, np.abs(u).sum(), np.abs(w).sum()


@pytest.mark.parametrize("name", list(CASES))
def test_vapour(name):
    from paper_1408_3764_amd.box import Box
    n, L, rc, cm, ns, crowd = CASES[name]
    rng = np.random.default_rng(3)
    pos = _gas(n, L, crowd, rng)
    n = len(pos)
    sp = rng.integers(0, ns, n).astype(np.int32)
    eps, sig = workloads.lorentz_berthelot([1.0, 1.2, 0.9, 1.1][:ns], [1.0, 0.8, 1.1, 0.7][:ns])
    if ns > 1:
        eps[0, ns - 1] = eps[ns - 1, 0] = 0.0
    b = Box(pos, L, rc, eps=eps, sigma=sig, species=sp if ns > 1 else None, cell_m=cm, max_n=n + 1)
    U, W, each, g, de, ds, su, sw = _sums(pos, L, rc, eps, sig, sp)
    p = oracle.make_params(L, rc, eps=eps, sigma=sig)
    counts = np.bincount(sp, minlength=ns)
    t = b.total_energy()
    assert abs(t["U_pair"] - U) <= 1e-10 * su and t["U_tail"] == pytest.approx(oracle.tail_energy(counts, p), rel=1e-12)
    t = b.total_energy(per_particle=True)
    assert abs(t["U_pair"] - U) <= 1e-10 * su
    assert np.allclose(t["e"], each, rtol=0, atol=1e-10 * np.abs(each).max())
    assert abs(b.virial()["W"] - W) <= 1e-10 * sw
    out = b.backward()
    assert np.allclose(out["grad"], g, rtol=1e-7, atol=1e-7 * np.abs(g).max())
    assert np.array_equal(b.backward(params=False)["grad"], out["grad"])
    nn, V, x = np.outer(counts, counts), float(np.prod(L)), sig / rc
    te = 8 * np.pi / (3 * V) * nn * sig ** 3 * (x ** 9 / 3 - x ** 3)
    ts = 8 * np.pi / (3 * V) * nn * eps * sig ** 2 * (4 * x ** 9 - 6 * x ** 3)
    assert np.allclose(out["d_eps"], de + te, rtol=1e-7, atol=1e-7 * np.abs(de + te).max())
    assert np.allclose(out["d_sigma"], ds + ts, rtol=1e-7, atol=1e-7 * np.abs(ds + ts).max())
    # single particles, the crowd's among them, against the oracle
    for i in np.concatenate([rng.integers(0, n, 12), [n - 1]]):
        e, mag = oracle.position_energy(pos, p, pos[i], exclude=int(i), species=sp, point_species=int(sp[i]))
        assert abs(t["e"][i] - e) <= 1e-10 * max(mag, 1e-300)
        assert np.allclose(out["grad"][i], oracle.particle_gradient(pos, int(i), p, species=sp), rtol=1e-7, atol=1e-7)


def test_vapour_with_an_overlap():
    """Two particles in one place: +inf in the totals and in their energies alone, gradients finite."""
    from paper_1408_3764_amd.box import Box
    L = (132.0, 132.0, 132.0)
    pos = _gas(66000, L, 0, np.random.default_rng(4))
    pos[7] = pos[60000]
    b = Box(pos, L, 2.5, max_n=66001)
    assert np.isposinf(b.total_energy()["U_pair"]) and np.isposinf(b.virial()["W"])
    assert np.array_equal(np.nonzero(np.isinf(b.total_energy(per_particle=True)["e"]))[0], [7, 60000])
    assert np.isfinite(b.backward()["grad"]).all()
