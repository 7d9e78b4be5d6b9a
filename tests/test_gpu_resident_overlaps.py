"""The LDS-held chain where a move's position lies on a particle that an earlier move of its round takes
away: the overlap's pair term (1e18 and more) is then not part of the move's sums, whose digits are all
there.  Every move's energy and virial change against the oracle's, to 1e-10 of the magnitudes that are
part of them."""
import numpy as np
import pytest

import oracle
from helpers import assert_du
from paper_1408_3764_amd import workloads

pytestmark = pytest.mark.gpu

KINDS = {"deletion, insertion": (2, 1), "deletion, displacement": (2, 0), "displacement, insertion": (0, 1),
         "displacement, displacement": (0, 0)}
N, L, T, MU = 90, 6.2, 1e3, -5e4      # deletions are accepted, insertions are not, one displacement in two is


def _params(L, n=N):
    wb = workloads.random_box(n, L, rc=2.5, T=T, seed=5, mu=MU)
    return wb, oracle.make_params(wb.L, 2.5, beta=wb.beta, mu=MU)


def _start(seed, kinds, last):
    """Positions whose moves j < k <= last of this seed are of these kinds, k's new position 0.03 from the
    particle j takes away; None if the seed's draws are not such, or j is not accepted."""
    wb, p = _params(L)
    draws = [oracle.move_draws(seed, m) for m in range(last + 1)]
    types = [0 if u[0] < 1.0 / 3.0 else (2 if u[1] < 0.5 else 1) for u in draws]
    picks = [oracle.pick(u[2], u[7], N) for u in draws]
    for j in range(last):
        for k in range(j + 1, last + 1):
            if (types[j], types[k]) != kinds or picks[j] == picks[k] or 1 in types[:j] or 2 in types[:j]:
                continue
            pos = wb.pos.copy()
            q = np.array(draws[k][4:7])
            new = q * L if types[k] == 1 else np.mod(pos[picks[k]] + 0.3 * (2.0 * q - 1.0), L)
            pos[picks[j]] = np.mod(new + np.array([0.03, 0.0, 0.0]), L)
            _, _, log = oracle.chain(pos, last + 1, p, seed=seed, max_n=N + 40)
            if log["accepted"][j] and int(log["index"][j]) == picks[j] and log["sumabs"][k] < 1e9 and (
                    types[k] == 1 or int(log["index"][k]) == picks[k]):
                return pos
    return None


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("kinds", list(KINDS))
def test_overlap_with_a_particle_taken_away(kinds, waves):
    from paper_1408_3764_amd.box import Box
    found = 0
    for seed in range(3000):
        pos = _start(seed, KINDS[kinds], waves - 1)
        if pos is None:
            continue
        wb, p = _params(L)
        b = Box(pos, wb.L, 2.5, beta=wb.beta, mu=MU, max_n=N + 40, cell_cap=64, seed=seed)
        b.set_launch(waves, -3)
        b.total_energy()
        _, log = b.step(16, counter0=0, log=True)
        _, _, olog = oracle.chain(pos, 16, p, seed=seed, max_n=N + 40)
        for f in ("type", "index", "accepted"):
            assert np.array_equal(log[f], olog[f]), (seed, f)
        assert_du(log["dU_pair"], olog["dU_pair"], olog["sumabs"], "dU, seed %d" % seed)
        assert_du(log["dW_pair"], olog["dW_pair"], olog["wsumabs"], "dW, seed %d" % seed)
        b.close()
        found += 1
        if found == 6:
            break
    assert found == 6


@pytest.mark.parametrize("waves", [4, 8])
@pytest.mark.parametrize("n,L,T,mu", [(120, 6.5, 1e9, 0.0), (6, 5.0, 1e9, -3e9), (2100, 14.0, 1e9, 0.0)])
def test_overlaps_come_and_go(n, L, T, mu, waves):
    """So hot that overlaps are accepted: many particles, few (most moves of a round on the same ones), and
    more than the LDS copy holds."""
    from paper_1408_3764_amd.box import Box
    wb = workloads.random_box(n, L, rc=2.5, T=T, seed=77, mu=mu)
    moves, max_n = 600, n + 800
    p = oracle.make_params(wb.L, 2.5, beta=wb.beta, mu=mu)
    b = Box.from_workload(wb, max_n=max_n, cell_cap=256)
    b.set_launch(waves, -3)
    b.total_energy()
    _, log = b.step(moves, counter0=0, log=True)
    pos, _, olog = oracle.chain(wb.pos, moves, p, seed=wb.seed, max_n=max_n)
    for f in ("type", "index", "accepted", "flags"):
        assert np.array_equal(log[f], olog[f]), f
    some = (olog["flags"] & 1) == 0
    assert_du(log["dU_pair"][some], olog["dU_pair"][some], olog["sumabs"][some], "dU")
    assert_du(log["dW_pair"][some], olog["dW_pair"][some], olog["wsumabs"][some], "dW")
    assert np.array_equal(b.particles()[0], pos)
