"""Timed cases: the work a program gives this library, through its public entry points.

Six kinds of call:

chain    one launch of a single box's Markov chain from a checkpoint, and the checkpoint after it
         (Box.restore, Box.step, gcmc_export_state): single boxes of a few hundred to 1.5 million
         particles, each with the launch shape its tuner picks
batch    one launch of many boxes, each on its own chain (Batch.step)
measure  the total energy (optionally every particle's) and the virial pressure of a
         configuration, as taken between launches
fit      one step of force-field fitting or force evaluation: the differentiable total energy at
         given positions and tables, and its gradients (lj_energy forward and backward)
trials   energy and virial changes of trial moves given by the host (Widom insertions,
         host-driven Monte Carlo): Box.delta_energy
volume   a rejected volume move: the box scaled, its energies read, and scaled back (Box.rescale)

Sizes are those of workloads.py (small, large, slab, batched, mixture, the size and cutoff
studies); configurations are jittered lattices with random vacancies at the same densities, which
are made in a fraction of a second at any size.
"""
import math

import numpy as np
import torch

from paper_1408_3764_amd import _lib, workloads
from paper_1408_3764_amd._lib import COUNTER_CONTINUE
from paper_1408_3764_amd.autograd import lj_energy
from paper_1408_3764_amd.box import Batch, Box, make_moves

MU = -3.0
MIX_SIGMA, MIX_EPS = [1.0, 1.2, 0.9, 1.1], [1.0, 0.8, 1.1, 0.9]   # per species, mixed by Lorentz-Berthelot


def listed():
    return [
        # the smallest box of the size study: the whole box held in LDS for the launch
        {"name": "chain-512", "kind": "chain", "n": 512, "rho": 0.67, "rc": 2.5, "T": 1.2, "moves": 1000,
         "waves": 8, "rows": -3, "cells": 1, "slab": False},
        # the small workload: 4,000 particles, 1,000 moves
        {"name": "chain-4000", "kind": "chain", "n": 4000, "rho": 0.5, "rc": 2.5, "T": 1.2, "moves": 1000,
         "waves": 8, "rows": 0, "cells": 1, "slab": False},
        # a cutoff of 4.25 on microcells (the cutoff study's largest cutoff)
        {"name": "chain-87296-rc4.25", "kind": "chain", "n": 87296, "rho": 0.666, "rc": 4.25, "T": 1.2, "moves": 4000,
         "waves": 8, "rows": 0, "cells": 2, "slab": False},
        # the headline workload: a liquid slab in its vapour, 1.5 million particles
        {"name": "chain-slab-1500000", "kind": "chain", "n": 1500000, "rho": 0.8, "rc": 2.5, "T": 0.85,
         "moves": 10000, "waves": 8, "rows": 0, "cells": 1, "slab": True},
        # many independent boxes on one GPU
        {"name": "batch-512", "kind": "batch", "boxes": 512, "n_min": 128, "n_max": 32768, "moves": 1000},
        # averages of a small box between launches: latency and launches
        {"name": "measure-4000", "kind": "measure", "n": 4000, "rho": 0.5, "rc": 2.5, "species": 1, "each": False},
        # the mixture workload's energy and pressure
        {"name": "measure-mix-262144", "kind": "measure", "n": 262144, "rho": 0.6, "rc": 3.0, "species": 2,
         "each": False},
        # a small force-field fit
        {"name": "fit-500", "kind": "fit", "n": 500, "rho": 0.376, "rc": 3.0, "species": 2},
        # the mixture workload's forces and parameter gradients
        {"name": "fit-mix-262144", "kind": "fit", "n": 262144, "rho": 0.6, "rc": 3.0, "species": 2},
        # one host-driven move at a time
        {"name": "trials-4000-1", "kind": "trials", "n": 4000, "rho": 0.5, "rc": 2.5, "species": 1, "trials": 1},
        # test-particle insertions and trial moves against the large workload's box
        {"name": "trials-262144-16384", "kind": "trials", "n": 262144, "rho": 0.7, "rc": 3.0, "species": 1,
         "trials": 16384},
        # volume moves of a mid-sized box
        {"name": "volume-32768", "kind": "volume", "n": 32768, "rho": 0.67, "rc": 2.5},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["chain", "chain", "batch", "measure", "measure", "fit", "fit", "trials", "trials", "volume"])
    rho = round(rng.uniform(0.3, 0.8), 3)
    if kind == "batch":
        return {"kind": kind, "boxes": _log_int(rng, 8, 512), "n_min": 128, "n_max": _log_int(rng, 1024, 32768),
                "moves": _log_int(rng, 100, 1000)}
    if kind == "chain":
        n = _log_int(rng, 200, 1000000)
        slab = n >= 50000 and rng.random() < 0.3
        rc = 2.5 if slab or n < 2000 else round(rng.uniform(2.5, 4.25), 2)
        waves, rows, cells = 8, 0, 1
        if n <= 1400:
            waves, rows = rng.choice([4, 8]), -3
        elif rc >= 3.5:
            cells = 2
        return {"kind": kind, "n": n, "rho": 0.8 if slab else rho, "rc": rc, "T": round(rng.uniform(0.85, 1.5), 2),
                "moves": _log_int(rng, 100, 10000), "waves": waves, "rows": rows, "cells": cells, "slab": slab}
    if kind == "volume":
        return {"kind": kind, "n": _log_int(rng, 500, 262144), "rho": rho, "rc": 2.5}
    species = rng.choice([1, 1, 2, 3])
    rc = round(rng.uniform(2.5, 3.5), 2) if species == 1 else 3.0
    case = {"kind": kind, "n": _log_int(rng, 400, 262144), "rho": rho if species == 1 else min(rho, 0.6), "rc": rc,
            "species": species}
    if kind == "measure":
        case["each"] = rng.random() < 0.4
    if kind == "trials":
        case["trials"] = _log_int(rng, 1, 16384)
    return case


# ------------------------------------------------------------- inputs
def _edges(case):
    if case.get("slab"):
        a = (case["n"] / (2.0 * case["rho"] + 2.0 * 0.02)) ** (1.0 / 3.0)
        return np.array([a, a, 4.0 * a])
    return np.full(3, float(np.cbrt(case["n"] / case["rho"])))


def _grid_m(L, rc):
    return [max(3, int(math.floor(v / rc))) for v in L]


def _lattice(rng, n, L, lo, hi):
    """n points on randomly chosen sites of a cubic lattice filling [lo, hi), jittered as far as
    neighbouring points then keep about 0.9 apart."""
    ext = hi - lo
    s = (float(np.prod(ext)) / (1.04 * n)) ** (1.0 / 3.0)
    m = np.maximum(1, np.ceil(ext / s)).astype(np.int64)
    sites = rng.permutation(int(np.prod(m)))[:n]
    ijk = np.stack([sites % m[0], sites // m[0] % m[1], sites // (m[0] * m[1])], axis=1)
    step = ext / m
    jitter = 0.5 * np.clip(step - 0.9, 0.02, None)
    pts = lo + (ijk + 0.5) * step + rng.uniform(-1.0, 1.0, (n, 3)) * jitter
    return np.clip(pts, 0.0, np.nextafter(L, 0.0))


def _positions(case, rng):
    L, n = _edges(case), case["n"]
    if not case.get("slab"):
        return _lattice(rng, n, L, np.zeros(3), L.copy()), L
    a = L[0]
    n_l = min(n, int(round(2.0 * case["rho"] * a ** 3)))
    n_v = (n - n_l) // 2
    parts = [_lattice(rng, n_l, L, np.array([0, 0, a]), np.array([a, a, 3 * a])),
             _lattice(rng, n_v, L, np.array([0, 0, 1.0]), np.array([a, a, a - 1.0])),
             _lattice(rng, n - n_l - n_v, L, np.array([0, 0, 3 * a + 1.0]), np.array([a, a, 4 * a - 1.0]))]
    pos = np.concatenate(parts)
    return pos[rng.permutation(n)], L


def _tables(ns):
    if ns == 1:
        return np.ones((1, 1)), np.ones((1, 1))
    return workloads.lorentz_berthelot(MIX_SIGMA[:ns], MIX_EPS[:ns])


def _make_moves(case, pos, L, species, rng):
    m = case["trials"]
    types = rng.integers(0, 3, m)
    index = rng.integers(0, case["n"], m)
    near = np.mod(pos[index] + rng.uniform(-0.3, 0.3, (m, 3)), L)
    pts = np.where(types[:, None] == 1, rng.random((m, 3)) * L, near)
    pts = np.clip(pts, 0.0, np.nextafter(L, 0.0))
    return make_moves(types, index, pts, rng.integers(0, case["species"], m))


def _inputs(case, seed):
    rng = np.random.Generator(np.random.PCG64(seed))
    pos, L = _positions(case, rng)
    ns = case.get("species", 1)
    species = rng.integers(0, ns, case["n"]).astype(np.int32) if ns > 1 else None
    return pos, L, species, rng


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        return _prepare_batch(case, seed)
    pos, L, species, rng = _inputs(case, seed)
    eps, sigma = _tables(case.get("species", 1))
    kw = {}
    if kind == "chain":
        kw = {"beta": 1.0 / case["T"], "mu": MU, "max_n": case["n"] + case["moves"],
              "cell_m": None if case["cells"] == 1 else [case["cells"] * m for m in _grid_m(L, case["rc"])]}
    if kind == "volume":
        kw = {"max_n": case["n"] + 1}
    box = Box(pos, L, case["rc"], eps=eps, sigma=sigma, species=species, seed=seed, **kw)
    state = {"case": case, "box": box}
    if kind == "chain":
        box.set_launch(case["waves"], case["rows"])
        box.total_energy()
        box.virial()
        state["snap"] = box.snapshot()
        state["after"] = [torch.zeros(box.max_n, dtype=torch.float64, device=box.device) for _ in range(3)]
    elif kind == "measure":
        state["n"] = case["n"]
    elif kind == "fit":
        dev = box.device
        state["pos"] = torch.tensor(pos, dtype=torch.float64, device=dev, requires_grad=True)
        state["eps"] = torch.tensor(eps, dtype=torch.float64, device=dev, requires_grad=True)
        state["sigma"] = torch.tensor(sigma, dtype=torch.float64, device=dev, requires_grad=True)
    elif kind == "trials":
        state["moves"] = _make_moves(case, pos, L, species, rng)
    elif kind == "volume":
        state["edges"] = (L * 1.01, L)
        state["after"] = [torch.zeros(box.max_n, dtype=torch.float64, device=box.device) for _ in range(3)]
    return state


def _prepare_batch(case, seed):
    """Boxes of log-uniform sizes.  The chains run on from pass to pass, so every box has room (cells
    and particles) for the densities the chemical potential leads to."""
    rng = np.random.Generator(np.random.PCG64(seed))
    boxes = []
    for k in range(case["boxes"]):
        n = int(round(math.exp(rng.uniform(math.log(case["n_min"]), math.log(case["n_max"])))))
        rho, T = rng.uniform(0.3, 0.8), rng.uniform(0.9, 1.5)
        one = {"n": n, "rho": rho}
        pos, L = _positions(one, rng)
        s = L[0] / max(3, int(math.floor(L[0] / 2.5)))
        b = Box(pos, L, 2.5, beta=1.0 / T, mu=MU, max_n=int(1.1 * n / rho) + 64, cell_cap=4 * int(0.4 * s ** 3 + 4),
                seed=seed, box_id=k)
        b.set_launch(4, -3 if n <= 1536 else 0)
        b.total_energy()
        b.virial()
        boxes.append(b)
    return {"case": case, "boxes": boxes, "batch": Batch(boxes)}


# --------------------------------------------------------------- a pass
_COUNTS = ("attempts", "accepts", "n", "moves_done", "stencils", "candidates", "pair_evals", "in_cutoff", "error")
_VALUES = ("u_pair", "u_tail", "w_pair", "sum_n", "sum_u", "sum_w", "sum_n2", "avg_n", "avg_u", "avg_p")


def _stats(st):
    return {"counts": {k: np.asarray(st[k]).astype(np.int64) for k in _COUNTS},
            "values": {k: np.asarray(st[k], dtype=np.float64) for k in _VALUES}}


def _energies(d):
    return np.array([d["U_pair"], d["U_tail"], d["U_pair_old"], d["U_tail_old"]])


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "batch":
        return _stats(state["batch"].step(case["moves"], counter0=COUNTER_CONTINUE))
    box = state["box"]
    if kind == "chain":
        box.restore(state["snap"])
        st, _ = box.step(case["moves"], counter0=COUNTER_CONTINUE)
        x, y, z = state["after"]   # the program's checkpoint arrays (max_n long)
        ck = _lib.gcmc_export_state(box.handle, x, y, z, None, box.max_n, box.stream)
        return {"stats": _stats(st), "x": x, "y": y, "z": z, "n": int(ck.n), "counter": int(ck.counter)}
    if kind == "measure":
        w = torch.empty(2, dtype=torch.float64, device=box.device)
        if case["each"]:
            u = torch.empty(2, dtype=torch.float64, device=box.device)
            e = torch.empty(state["n"], dtype=torch.float64, device=box.device)
            _lib.gcmc_total_energy(box.handle, 0, u, e, box.stream)
            _lib.gcmc_virial(box.handle, w, box.stream)
            return {"U": u, "WP": w, "e": e}
        u = box.total_energy_device()
        _lib.gcmc_virial(box.handle, w, box.stream)
        return {"U": u, "WP": w}
    if kind == "fit":
        u = lj_energy(state["pos"], state["eps"], state["sigma"], box)
        g, de, ds = torch.autograd.grad(u, (state["pos"], state["eps"], state["sigma"]))
        return {"U": u.detach(), "pos": g, "eps": de, "sigma": ds}
    if kind == "trials":
        du, dt, dw = box.delta_energy(state["moves"], virial=True)
        return {"dU": du, "dU_tail": dt, "dW": dw}
    up = box.rescale(state["edges"][0])
    back = box.rescale(state["edges"][1])
    x, y, z = state["after"]
    ck = _lib.gcmc_export_state(box.handle, x, y, z, None, box.max_n, box.stream)
    return {"up": _energies(up), "back": _energies(back), "x": x, "y": y, "z": z, "n": int(ck.n)}


# ------------------------------------------------------------ least work
def _sphere(case):
    """Mean number of particles within the cutoff of a point (the box's own number at most)."""
    return min(float(case["n"]), case["rho"] * 4.0 / 3.0 * math.pi * case["rc"] ** 3)


def work(case):
    """Per pair inside the cutoff: 8 operations for the squared distance and 12 for energy and
    virial (18 for the gradient terms); per trial position, the particles within the cutoff once."""
    kind = case["kind"]
    if kind == "batch":
        mean_n = (case["n_max"] - case["n_min"]) / math.log(case["n_max"] / case["n_min"])
        near = 0.55 * 4.0 / 3.0 * math.pi * 2.5 ** 3
        moves = case["boxes"] * case["moves"]
        return {"bytes": moves * (4.0 / 3.0) * near * 24.0 + case["boxes"] * min(mean_n, case["moves"]) * 32.0,
                "flops": moves * (4.0 / 3.0) * near * 20.0}
    n, near = case["n"], _sphere(case)
    if kind == "chain":
        moved = case["moves"] * (4.0 / 3.0) * near
        return {"bytes": moved * 24.0 + 4.0 * 28.0 * n, "flops": moved * 20.0}
    if kind == "measure":
        extra = 8.0 * n if case["each"] else 0.0
        return {"bytes": 28.0 * n + extra, "flops": 0.5 * n * near * (8.0 + 12.0)}
    if kind == "fit":
        return {"bytes": 28.0 * n + 24.0 * n, "flops": 0.5 * n * near * (8.0 + 12.0 + 18.0)}
    if kind == "trials":
        moved = case["trials"] * (4.0 / 3.0) * near
        return {"bytes": case["trials"] * (40.0 + 24.0) + min(moved, n) * 24.0, "flops": moved * 20.0}
    return {"bytes": 6.0 * 24.0 * n, "flops": 3.0 * 0.5 * n * near * 20.0}


# -------------------------------------------- plain 64-bit reference values
def _window_pairs(pos, L, rc, chunk=2048):
    """Ordered pairs closer than rc, a chunk of first particles at a time: (i, j, d = r_j - r_i at
    minimum image, r^2).  The particles are sorted by z, and a chunk meets only those within rc of
    its z range."""
    order = torch.argsort(pos[:, 2])
    p = pos[order]
    n = p.shape[0]
    z = p[:, 2].contiguous()
    for a in range(0, n, chunk):
        b = min(n, a + chunk)
        lo, hi = float(z[a]) - rc, float(z[b - 1]) + rc
        keep = torch.zeros(n, dtype=torch.bool, device=p.device)
        for s in (-float(L[2]), 0.0, float(L[2])):
            keep |= (z + s >= lo) & (z + s <= hi)
        near = torch.nonzero(keep)[:, 0]
        q = p[near]
        step = max(1, int(4e7) // max(1, len(near)))
        for c in range(a, b, step):
            e = min(b, c + step)
            d = q[None, :, :] - p[c:e, None, :]
            d = d - L * torch.round(d / L)
            r2 = (d * d).sum(-1)
            i, j = torch.nonzero((r2 < rc * rc) & (near[None, :] != torch.arange(c, e, device=p.device)[:, None]),
                                 as_tuple=True)
            yield order[c + i], order[near[j]], d[i, j], r2[i, j]


def _tail(counts, V, rc, eps, sig):
    """Energy and pressure of the full potential beyond rc, and the energy's table derivatives."""
    nn = np.outer(counts, counts)
    x = sig / rc
    k = 8.0 * math.pi / (3.0 * V) * nn
    u = k * eps * sig ** 3 * (x ** 9 / 3.0 - x ** 3)
    p = 16.0 * math.pi / (3.0 * V * V) * nn * eps * sig ** 3 * (2.0 / 3.0 * x ** 9 - x ** 3)
    return u.sum(), p.sum(), k * sig ** 3 * (x ** 9 / 3.0 - x ** 3), k * eps * sig ** 2 * (4.0 * x ** 9 - 6.0 * x ** 3)


def _totals(pos, L, species, rc, ns, grad):
    """Pair sums of a configuration by plain torch in 64 bits."""
    dev = torch.device("cuda")
    eps, sig = _tables(ns)
    p = torch.tensor(pos, dtype=torch.float64, device=dev)
    Lt = torch.tensor(L, dtype=torch.float64, device=dev)
    sp = torch.zeros(len(pos), dtype=torch.int64, device=dev) if species is None else torch.tensor(
        species, dtype=torch.int64, device=dev)
    et = torch.tensor(eps, dtype=torch.float64, device=dev).reshape(-1)
    st = torch.tensor(sig, dtype=torch.float64, device=dev).reshape(-1)
    e = torch.zeros(len(pos), dtype=torch.float64, device=dev)
    g = torch.zeros_like(p) if grad else None
    w = torch.zeros((), dtype=torch.float64, device=dev)
    de, ds = torch.zeros(ns * ns, dtype=torch.float64, device=dev), torch.zeros(ns * ns, dtype=torch.float64, device=dev)
    for i, j, d, r2 in _window_pairs(p, Lt, rc):
        q = sp[i] * ns + sp[j]
        ep, s6 = et[q], (st[q] ** 2 / r2) ** 3
        s12 = s6 * s6
        e.index_add_(0, i, 4.0 * ep * (s12 - s6))
        w += (12.0 * ep * (2.0 * s12 - s6)).sum()
        if grad:
            g.index_add_(0, i, (24.0 * ep * (2.0 * s12 - s6) / r2)[:, None] * d)
            de.index_add_(0, q, 2.0 * (s12 - s6))
            ds.index_add_(0, q, 2.0 * ep / st[q] * (12.0 * s12 - 6.0 * s6))
    counts = np.array([int((sp == a).sum()) for a in range(ns)], dtype=np.float64)
    V = float(np.prod(L))
    ut, pt, te, ts = _tail(counts, V, rc, eps, sig)
    out = {"U": np.array([0.5 * float(e.sum()), ut]), "W": float(w), "e": e.cpu().numpy(),
           "P": len(pos) / V + float(w) / (3.0 * V) + pt}
    if grad:
        out.update(grad=g.cpu().numpy(), d_eps=de.cpu().numpy().reshape(ns, ns) + te,
                   d_sigma=ds.cpu().numpy().reshape(ns, ns) + ts)
    return out


def _trial_values(case, pos, L, species, moves):
    dev = torch.device("cuda")
    ns, rc = case["species"], case["rc"]
    eps, sig = _tables(ns)
    p, Lt = torch.tensor(pos, dtype=torch.float64, device=dev), torch.tensor(L, dtype=torch.float64, device=dev)
    sp = torch.zeros(len(pos), dtype=torch.int64, device=dev) if species is None else torch.tensor(
        species, dtype=torch.int64, device=dev)
    et = torch.tensor(eps, dtype=torch.float64, device=dev).reshape(-1)
    st = torch.tensor(sig, dtype=torch.float64, device=dev).reshape(-1)
    kind = torch.tensor(moves["type"].astype(np.int64), device=dev)
    index = torch.tensor(moves["index"].astype(np.int64), device=dev)
    new = torch.tensor(np.stack([moves["x"], moves["y"], moves["z"]], axis=1), device=dev)
    own = torch.where(kind == 1, torch.tensor(moves["species"].astype(np.int64), device=dev), sp[index])
    skip = torch.where(kind == 1, -1, index)

    def sums(at):
        u, w = torch.zeros(len(at), dtype=torch.float64, device=dev), torch.zeros(len(at), dtype=torch.float64, device=dev)
        step = max(1, int(4e7) // len(pos))
        ids = torch.arange(len(pos), device=dev)
        for c in range(0, len(at), step):
            d = p[None] - at[c:c + step, None]
            d = d - Lt * torch.round(d / Lt)
            r2 = (d * d).sum(-1)
            i, j = torch.nonzero((r2 < rc * rc) & (ids[None] != skip[c:c + step, None]), as_tuple=True)
            q = own[c + i] * ns + sp[j]
            s6 = (st[q] ** 2 / r2[i, j]) ** 3
            u.index_add_(0, c + i, 4.0 * et[q] * (s6 * s6 - s6))
            w.index_add_(0, c + i, 24.0 * et[q] * (2.0 * s6 * s6 - s6))
        return u, w

    un, wn = sums(new)
    uo, wo = sums(p[index])
    du = torch.where(kind == 0, un - uo, torch.where(kind == 1, un, -uo))
    dw = torch.where(kind == 0, wn - wo, torch.where(kind == 1, wn, -wo))
    counts = np.array([int((sp == a).sum()) for a in range(ns)], dtype=np.float64)
    x = sig / rc
    k = 8.0 * math.pi / (3.0 * float(np.prod(L))) * eps * sig ** 3 * (x ** 9 / 3.0 - x ** 3)
    o = own.cpu().numpy()
    lin, sq = 2.0 * (k[o] @ counts), k[o, o]
    dt = np.where(moves["type"] == 0, 0.0, np.where(moves["type"] == 1, lin + sq, -lin + sq))
    return {"dU": du.cpu().numpy(), "dU_tail": dt, "dW": dw.cpu().numpy()}


def exact(case, seed):
    kind = case["kind"]
    if kind in ("chain", "batch"):
        return None   # a chain's values follow from its decisions; those are compared as whole numbers
    pos, L, species, rng = _inputs(case, seed)
    if kind == "trials":
        if case["trials"] * case["n"] > 6e9:
            return None
        return _trial_values(case, pos, L, species, _make_moves(case, pos, L, species, rng))
    if kind == "volume":
        up_L = L * 1.01
        t0 = _totals(pos, L, None, case["rc"], 1, False)["U"]
        big = pos * (up_L / L)
        t1 = _totals(big, up_L, None, case["rc"], 1, False)["U"]
        small = big * (L / up_L)
        t2 = _totals(small, L, None, case["rc"], 1, False)["U"]

        x, y, z = (np.append(small[:, a], 0.0) for a in range(3))   # the arrays hold max_n = n + 1
        return {"up": np.concatenate([t1, t0]), "back": np.concatenate([t2, t1]), "x": x, "y": y, "z": z}
    t = _totals(pos, L, species, case["rc"], case["species"], kind == "fit")
    if kind == "fit":
        return {"U": np.array(t["U"][0] + t["U"][1]), "pos": t["grad"], "eps": t["d_eps"], "sigma": t["d_sigma"]}
    out = {"U": t["U"], "WP": np.array([t["W"], t["P"]])}
    if case["each"]:
        out["e"] = t["e"]
    return out
