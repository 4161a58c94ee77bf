"""Timed cases of the library's public entry points on one GPU.

Four kinds of work make up the range a program has the library do:

  eval   Tissue.energy_forces (energy, forces, max |F|) on one tissue of 64 to
         10^6 cells in each precision mode, uniform or per-cell parameters;
  relax  gradient descent: Tissue.relax on one tissue, Batch.relax on many
         (equal or mixed sizes), with and without T1 exchanges.  A pass takes
         `steps` more steps from where the last one stopped, as a program
         that watches a long relaxation calls it;
  solve  derivatives of an outer cost at a settled state: Tissue.param_grad
         (adjoint by CG or MINRES), Tissue.param_sens (forward), and their
         batched form Batch.param_grad;
  ep     Batch.param_grad by centred equilibrium propagation, a fixed number
         of nudged steps towards target positions;
  fit    one outer step of the bilevel loop: autograd.equilibrium forward
         (relaxation with T1 from the previous equilibrium) and backward
         (adjoint).

Tissues relaxed with T1 start at random Voronoi tilings (as the rigidity
study and the batched workload do); the others, and the settled states, are
built here from evenly spread seeds, the latter by plain torch steps, so they
do not depend on the library.
Parameters follow the library's workloads: K_A = A0 = K_P = 1, P0 around
3.75, line tensions U[0.05, 0.15] (settled states: U[0.08, 0.12]).
"""
from __future__ import annotations

import functools
import math

import numpy as np
import torch

from paper_2604_06896_amd import tissue_gen as g
from paper_2604_06896_amd import vtx as V
from paper_2604_06896_amd.autograd import equilibrium

DEV = "cuda"
F64 = torch.float64


# --------------------------------------------------------------------- cases
def listed():
    return [
        # one evaluation of a small tissue (an optimiser or a test harness
        # calling it in a loop): latency
        {"name": "eval_f64_100", "kind": "eval", "mode": "f64", "patch": 100, "rep": 1,
         "hetero": True},
        # a mid-size tissue with per-cell parameters
        {"name": "eval_mixed_10k", "kind": "eval", "mode": "mixed", "patch": 9973, "rep": 1,
         "hetero": True},
        # the throughput workload: 10^6 cells (8 x 8 copies of a 15625-cell
        # patch, every vertex displaced on its own)
        {"name": "eval_f32_1m", "kind": "eval", "mode": "f32", "patch": 15625, "rep": 8,
         "hetero": False},
        # a single small simulation with exchanges
        {"name": "relax_f64_100_t1", "kind": "relax", "mode": "f64", "cells": 100, "tissues": 1,
         "cells_max": 100, "t1": True, "steps": 1000},
        # a single simulation of ordinary size with exchanges
        {"name": "relax_mixed_10k_t1", "kind": "relax", "mode": "mixed", "cells": 10000,
         "tissues": 1, "cells_max": 10000, "t1": True, "steps": 1000},
        # many small tissues of one size (one value of the rigidity study)
        {"name": "batch_mixed_100x100_t1", "kind": "relax", "mode": "mixed", "cells": 100,
         "tissues": 100, "cells_max": 100, "t1": True, "steps": 1000},
        # the batched workload: 512 tissues of 64 to 4096 cells
        {"name": "batch_mixed_512_t1", "kind": "relax", "mode": "mixed", "cells": 64,
         "tissues": 512, "cells_max": 4096, "t1": True, "steps": 200},
        # one gradient of a large tissue
        {"name": "adjoint_f64_20k", "kind": "solve", "how": "adjoint", "theta": "lambda",
         "cells": 20000, "tissues": 1},
        # one forward derivative at the inverse workload's size
        {"name": "sens_f64_1000", "kind": "solve", "how": "sens", "theta": "P0", "cells": 1000,
         "tissues": 1},
        # the inverse workload: gradients of 64 tissues of 1000 cells
        {"name": "batch_adjoint_64x1000", "kind": "solve", "how": "adjoint", "theta": "lambda",
         "cells": 1000, "tissues": 64},
        # the same by equilibrium propagation (a fixed number of steps)
        {"name": "batch_ep_64x1000", "kind": "ep", "theta": "lambda", "cells": 1000,
         "tissues": 64, "steps": 1000},
        # one outer step of a parameter fit
        {"name": "fit_f64_20", "kind": "fit", "cells": 20},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["eval", "eval", "relax", "relax", "batch", "batch", "solve", "solve",
                       "ep", "fit"])
    if kind == "eval":
        n = _log_int(rng, 64, 1000000)
        rep = 1 if n <= 20000 else int(math.ceil(math.sqrt(n / 20000)))
        return {"kind": "eval", "mode": rng.choice(["f32", "mixed", "f64"]) if n < 400000
                else "f32", "patch": max(64, n // rep ** 2), "rep": rep,
                "hetero": rng.random() < 0.5}
    if kind == "relax":
        n = _log_int(rng, 20, 10000)
        return {"kind": "relax", "mode": rng.choice(["f32", "mixed", "f64"]), "cells": n,
                "tissues": 1, "cells_max": n, "t1": rng.random() < 0.6,
                "steps": rng.randint(200, 1000)}
    if kind == "batch":
        lo = _log_int(rng, 20, 1000)
        hi = lo if rng.random() < 0.5 else min(4096, _log_int(rng, lo, 8 * lo))
        return {"kind": "relax", "mode": rng.choice(["mixed", "f64"]), "cells": lo,
                "tissues": max(2, min(256, _log_int(rng, 16000, 128000) // hi)),
                "cells_max": hi, "t1": rng.random() < 0.6, "steps": rng.randint(100, 400)}
    if kind == "solve":
        how = rng.choice(["adjoint", "adjoint", "sens", "minres"])
        theta = rng.choice(["lambda", "P0"])
        if how == "sens" or rng.random() < 0.5:
            return {"kind": "solve", "how": how, "theta": theta, "tissues": 1,
                    "cells": _log_int(rng, 60, 12000)}
        n = _log_int(rng, 60, 1600)
        return {"kind": "solve", "how": how, "theta": theta, "cells": n,
                "tissues": max(2, min(128, _log_int(rng, 4000, 64000) // n))}
    if kind == "ep":
        n = _log_int(rng, 60, 1000)
        return {"kind": "ep", "theta": rng.choice(["lambda", "P0"]), "cells": n,
                "tissues": max(2, min(60, _log_int(rng, 4000, 60000) // n)),
                "steps": rng.randint(300, 900)}
    return {"kind": "fit", "cells": rng.randint(16, 300)}


# ------------------------------------------------------------------- tissues
@functools.lru_cache(maxsize=64)
def _voronoi(n, variant):
    return g.random_tissue(n, rng=np.random.default_rng([n, variant]))


@functools.lru_cache(maxsize=64)
def _even(n, variant):
    """About n cells of even size: random seeds after 80 Lloyd steps (mostly
    six sides, a third with five or seven, and no edges short enough to
    collapse without T1).  Beyond 500 cells copies of a smaller tiling."""
    rep = int(math.ceil(math.sqrt(n / 500)))
    if rep > 1:
        return _replicate(_even(n // rep ** 2, variant), rep)
    L, rng = math.sqrt(n), np.random.default_rng([n, variant, 7])
    seeds = rng.uniform(0.0, L, size=(n, 2))
    for _ in range(80):
        t = g.periodic_voronoi(seeds, L, L)
        seeds = _Model([t]).centres(torch.as_tensor(t.X, device=DEV)).cpu().numpy() % L
    return g.periodic_voronoi(seeds, L, L)


def _replicate(t, k):
    """k x k copies of a periodic tissue as one periodic tissue, the copies
    along a Morton curve and the edges along the vertex order (as the
    generator numbers them)."""
    if k == 1:
        return t
    he, nv, nc = t.he.astype(np.int64), t.n_vert, t.n_cell
    nh, n_e = he.shape[0], he.shape[0] // 2
    ij = np.stack(np.meshgrid(np.arange(k), np.arange(k), indexing="ij"), -1).reshape(-1, 2)
    rank = np.empty(k * k, np.int64)
    rank[g.morton_order(ij + 0.5, k, k)] = np.arange(k * k)

    def at(ox, oy):  # copy that lies (ox, oy) from each copy, [k*k, ...], and its image
        x, y = ij[:, :1] + ox[None, :], ij[:, 1:] + oy[None, :]
        return rank[(x % k) * k + y % k], x // k, y // k

    inv = np.argsort(rank)

    def ident(q, copy):  # id of half-edges q whose source is in `copy`: an edge is numbered
        # with the copy its even half-edge starts in
        x = ij[inv[copy], 0] + he[q, g.HE_OX] * (q % 2)
        y = ij[inv[copy], 1] + he[q, g.HE_OY] * (q % 2)
        return 2 * (rank[(x % k) * k + y % k] * n_e + q // 2) + q % 2

    zero = np.zeros(nh, np.int64)
    here = at(zero, zero)[0]
    there, wx, wy = at(he[:, g.HE_OX], he[:, g.HE_OY])
    p = he[:, g.HE_PREV]
    before = at(-he[p, g.HE_OX], -he[p, g.HE_OY])[0]
    # offset of each half-edge's source from the first corner of its face
    walk_x, walk_y = zero.copy(), zero.copy()
    first = np.full(nc, -1, np.int64)
    first[he[::-1, g.HE_FACE]] = np.arange(nh)[::-1]
    h, cx, cy = first.copy(), np.zeros(nc, np.int64), np.zeros(nc, np.int64)
    for _ in range(int(np.bincount(he[:, g.HE_FACE]).max()) - 1):
        cx, cy = cx + he[h, g.HE_OX], cy + he[h, g.HE_OY]
        h = he[h, g.HE_NEXT]
        go = h != first
        cx[~go] = cy[~go] = 0
        walk_x[h[go]], walk_y[h[go]] = cx[go], cy[go]
    face = at(-walk_x, -walk_y)[0]
    hid = ident(np.arange(nh), here).ravel()
    out = np.empty((k * k * nh, 8), np.int64)
    out[hid, g.HE_PREV] = ident(p, before).ravel()
    out[hid, g.HE_NEXT] = ident(he[:, g.HE_NEXT], there).ravel()
    out[hid, g.HE_TWIN] = hid ^ 1
    out[hid, g.HE_SRC] = (here * nv + he[:, g.HE_SRC]).ravel()
    out[hid, g.HE_TGT] = (there * nv + he[:, g.HE_TGT]).ravel()
    out[hid, g.HE_FACE] = (face * nc + he[:, g.HE_FACE]).ravel()
    out[hid, g.HE_OX], out[hid, g.HE_OY] = wx.ravel(), wy.ravel()
    lo = np.minimum(out[0::2, g.HE_SRC], out[0::2, g.HE_TGT])
    hi = np.maximum(out[0::2, g.HE_SRC], out[0::2, g.HE_TGT])
    perm = np.lexsort((hi, lo))
    new = np.empty(k * k * n_e, np.int64)
    new[perm] = np.arange(k * k * n_e)
    out = out.reshape(-1, 2, 8)[perm].reshape(-1, 8)
    for col in (g.HE_PREV, g.HE_NEXT, g.HE_TWIN):
        out[:, col] = 2 * new[out[:, col] // 2] + out[:, col] % 2
    X = np.empty((k * k * nv, 2))
    for c in range(k * k):
        X[rank[c] * nv:(rank[c] + 1) * nv] = t.X + ij[c] * [t.Lx, t.Ly]
    return g.Tissue(out.astype(np.int32), X, k * t.Lx, k * t.Ly)


@functools.lru_cache(maxsize=4)
def _sheet(patch, rep):
    return _replicate(_voronoi(patch, 0), rep)


def _sizes(case):
    """Cells of each tissue of a relaxation case: `cells` to `cells_max`, at
    most 32 (without T1: 8) different tilings."""
    n, lo, hi = case["tissues"], case["cells"], case["cells_max"]
    rng = np.random.default_rng([n, lo, hi])
    pool = [(int(c), j) for j, c in enumerate(rng.integers(lo, hi + 1, size=min(n, 32 if case["t1"] else 8)))]
    return [pool[i % len(pool)] for i in range(n)]


def _gen(seed):
    q = torch.Generator(device=DEV)
    q.manual_seed(seed)
    return q


def _rand(q, n, lo, hi, dt):
    return lo + (hi - lo) * torch.rand(n, generator=q, device=DEV, dtype=dt)


def _shake(q, X, amount, dt):
    X = torch.as_tensor(X, dtype=F64, device=DEV)
    return (X + amount * torch.randn(X.shape, generator=q, device=DEV, dtype=F64)).to(dt)


# ------------------------------------------------- the model in plain torch
class _Model:
    """Energy, forces and derivatives of disjoint tissues in 64 bits, from
    their half-edge tables: every sum is a gather, so results repeat."""

    def __init__(self, ts):
        idx, sh, mask, nb, nsh, cells, edges, ends, esh = [], [], [], [], [], [], [], [], []
        v0 = c0 = e0 = 0
        width = max(int(np.bincount(t.he[:, g.HE_FACE]).max()) for t in ts)
        for t in ts:
            he = t.he.astype(np.int64)
            nh, nc, box = he.shape[0], t.n_cell, np.array([t.Lx, t.Ly])
            off = he[:, [g.HE_OX, g.HE_OY]]
            first = np.full(nc, -1, np.int64)
            first[he[::-1, g.HE_FACE]] = np.arange(nh)[::-1]
            I, S, K = np.empty((nc, width), np.int64), np.zeros((nc, width, 2)), np.zeros((nc, width), bool)
            h, w, live = first.copy(), np.zeros((nc, 2), np.int64), np.ones(nc, bool)
            for k in range(width):  # beyond its sides a row repeats corner 0
                I[:, k] = np.where(live, he[h, g.HE_SRC], I[:, 0])
                S[:, k] = np.where(live[:, None], w * box, 0.0)
                K[:, k] = live
                w, h = w + off[h], he[h, g.HE_NEXT]
                live &= h != first
            out = np.full(t.n_vert, -1, np.int64)
            out[he[::-1, g.HE_SRC]] = np.arange(nh)[::-1]
            star = [out]
            for _ in range(2):
                star.append(he[he[star[-1], g.HE_PREV], g.HE_TWIN])
            star = np.stack(star, 1)
            idx.append(I + v0); sh.append(S); mask.append(K)
            nb.append(he[star, g.HE_TGT] + v0); nsh.append(off[star] * box)
            cells.append(he[star, g.HE_FACE] + c0); edges.append(star // 2 + e0)
            ends.append(he[0::2][:, [g.HE_SRC, g.HE_TGT]] + v0); esh.append(off[0::2] * box)
            v0, c0, e0 = v0 + t.n_vert, c0 + nc, e0 + nh // 2
        wide = [np.pad(a, ((0, 0), (0, width - a.shape[1]))) for a in idx]
        self.idx, self.sh, self.mask, self.nb, self.nsh, self.cells, self.edges, self.ends, self.esh = (
            torch.as_tensor(np.concatenate(a), device=DEV)
            for a in (wide, sh, mask, nb, nsh, cells, edges, ends, esh))

    def cell(self, X):
        r = X[self.idx] + self.sh
        r = r - r[:, :1]
        q = torch.roll(r, -1, 1)
        A = 0.5 * (r[..., 0] * q[..., 1] - r[..., 1] * q[..., 0]).sum(1)
        d = q - r
        l2 = (d * d).sum(-1)
        P = torch.where(l2 > 0, torch.sqrt(torch.where(l2 > 0, l2, 1.0)), 0.0).sum(1)
        return A, P

    def centres(self, X):
        r = X[self.idx] + self.sh
        q = torch.roll(r, -1, 1)
        w = (r[..., 0] * q[..., 1] - r[..., 1] * q[..., 0])[..., None]
        return ((r + q) * w).sum(1) / (3.0 * w.sum(1))

    def pull(self, X, cA, cP, lam):
        """Force of per-cell coefficients (dE/dA, dE/dP) and edge tensions."""
        d = X[self.nb] + self.nsh - X[:, None]
        u = d / torch.sqrt((d * d).sum(-1, keepdim=True))
        a, p = cA[self.cells], cP[self.cells]
        T = lam[self.edges] + p + torch.roll(p, 1, 1)
        D = 0.5 * (a - torch.roll(a, 1, 1))
        R = torch.stack([d[..., 1], -d[..., 0]], -1)
        return (u * T[..., None] - R * D[..., None]).sum(1)

    def force(self, X, P0, lam):
        A, P = self.cell(X)
        return self.pull(X, 2 * (A - 1), 2 * (P - P0), lam)

    def lengths(self, X):
        d = X[self.ends[:, 1]] + self.esh - X[self.ends[:, 0]]
        return torch.sqrt((d * d).sum(-1)), d

    def energy(self, X, P0, lam):
        A, P = self.cell(X)
        return (A - 1) ** 2 + (P - P0) ** 2, lam * self.lengths(X)[0]

    def hess(self, X, P0, lam, v):
        """H v."""
        f = lambda x: self.force(x, P0, lam)  # noqa: E731
        return -torch.func.jvp(f, (X,), (v,))[1]


def _cg(m, X, P0, lam, b, n_t):
    """H x = P b of n_t tissues of one size, to rounding."""
    def per(a, c):  # the dot product of each tissue
        return (a * c).reshape(n_t, -1).sum(1)

    def spread(s):
        return s.repeat_interleave(b.shape[0] // n_t)[:, None]

    def centred(a):
        a = a.reshape(n_t, -1, 2)
        return (a - a.mean(1, keepdim=True)).reshape(-1, 2)

    r = centred(b)
    x, q, rr = torch.zeros_like(b), r.clone(), per(r, r)
    stop = 1e-29 * rr.max()
    for k in range(20000):
        Hq = m.hess(X, P0, lam, q)
        go = rr > stop
        al = torch.where(go, rr / per(q, Hq), 0.0)
        x, r = x + spread(al) * q, r - spread(al) * Hq
        rn = per(r, r)
        q = r + spread(torch.where(go, rn / rr, 0.0)) * q
        rr = rn
        if k % 32 == 31 and not bool((rr > stop).any()):
            break
    return centred(x)


def _settled(ts, X, P0, lam, steps=600):
    """Accelerated gradient descent (fixed topology) to a state near
    equilibrium."""
    m = _Model(ts)
    v = torch.zeros_like(X)
    for _ in range(steps):
        v = 0.95 * v + 0.006 * m.force(X + 0.95 * v, P0, lam)
        X = X + v
    return m, X


# ------------------------------------------------------------------- prepare
def _split(a, ns):
    return list(torch.split(a, ns))


def _solve_inputs(case, seed):
    """Settled tissues, their parameters, target positions and a direction,
    concatenated over the tissues."""
    q, n = _gen(seed), case["tissues"]
    ts = [_even(case["cells"], i % 4) for i in range(n)]
    nv, nc, ne = (sum(getattr(t, a) for t in ts) for a in ("n_vert", "n_cell", "n_edge"))
    lam = _rand(q, ne, 0.08, 0.12, F64)
    P0 = _rand(q, nc, 3.65, 3.75, F64)
    X = _shake(q, np.concatenate([t.X for t in ts]), 0.01, F64)
    m, X = _settled(ts, X, P0, lam)
    Xt = X + 0.05 * torch.randn(X.shape, generator=q, device=DEV, dtype=F64)
    d = torch.randn(ne if case.get("theta") != "P0" else nc, generator=q, device=DEV, dtype=F64)
    return ts, m, X, P0, lam, Xt, d / d.norm()


def _params(ts, P0, lam):
    return [V.Params(KA=1.0, A0=1.0, KP=1.0, P0=p, lam=x)
            for p, x in zip(_split(P0, [t.n_cell for t in ts]), _split(lam, [t.n_edge for t in ts]))]


def _eval_inputs(case, seed):
    t, q, dt = _sheet(case["patch"], case["rep"]), _gen(seed), V.pos_dtype(case["mode"])
    X = _shake(q, t.X, 0.01, dt)
    lam = _rand(q, t.n_edge, 0.05, 0.15, dt)
    P0 = _rand(q, t.n_cell, 3.6, 3.9, dt) if case["hetero"] else 3.75
    return t, X, P0, lam


def _relax_inputs(case, seed):
    q, dt = _gen(seed), V.pos_dtype(case["mode"])
    # (without T1 a random tiling's short edges collapse and never settle)
    ts = [(_voronoi if case["t1"] else _even)(*s) for s in _sizes(case)]
    X = _shake(q, np.concatenate([t.X for t in ts]), 0.005, dt)
    lam = _rand(q, sum(t.n_edge for t in ts), 0.05, 0.15, dt)
    P0 = _rand(q, sum(t.n_cell for t in ts), 3.6, 3.9, dt)
    return ts, X, P0, lam


def prepare(case, seed):
    kind = case["kind"]
    if kind == "eval":
        t, X, P0, lam = _eval_inputs(case, seed)
        return {"case": case, "T": V.Tissue.from_tissue(t), "X": X,
                "P": V.Params(KA=1.0, A0=1.0, KP=1.0, P0=P0, lam=lam)}
    if kind == "relax":
        ts, X, P0, lam = _relax_inputs(case, seed)
        Ts = [V.Tissue.from_tissue(t) for t in ts]
        return {"case": case, "Ts": Ts, "B": V.Batch(Ts) if len(Ts) > 1 else None, "X": X,
                "Xs": _split(X, [t.n_vert for t in ts]), "Ps": _params(ts, P0, lam),
                "opts": dict(eta=3e-3, tol=0.0, max_iter=case["steps"], t1_enable=case["t1"],
                             l_min=0.01)}
    if kind == "fit":
        ts, m, X, P0, lam, Xt, _ = _solve_inputs({"cells": case["cells"], "tissues": 1}, seed)
        theta = (lam + 0.01 * torch.randn(lam.shape, generator=_gen(seed + 1), device=DEV,
                                          dtype=F64)).requires_grad_()
        return {"case": case, "T": V.Tissue.from_tissue(ts[0]), "X": X, "Xt": Xt, "theta": theta,
                "P": V.Params(KA=1.0, A0=1.0, KP=1.0, P0=P0, lam=0.0),
                "box": torch.tensor([ts[0].Lx, ts[0].Ly], dtype=F64, device=DEV)}
    ts, m, X, P0, lam, Xt, d = _solve_inputs(case, seed)
    Ts = [V.Tissue.from_tissue(t) for t in ts]
    ns = [t.n_vert for t in ts]
    b = (X - Xt) / ns[0]
    return {"case": case, "Ts": Ts, "B": V.Batch(Ts) if len(Ts) > 1 else None, "Xs": _split(X, ns),
            "Xt": _split(Xt, ns), "b": _split(b, ns), "Ps": _params(ts, P0, lam), "d": d}


# ----------------------------------------------------------------------- run
def run(s):
    c = s["case"]
    kind = c["kind"]
    if kind == "eval":
        return s["T"].energy_forces(s["X"], s["P"], mode=c["mode"], want_maxf=True)
    if kind == "relax":
        if s["B"] is None:
            r = [s["Ts"][0].relax(s["X"], s["Ps"][0], mode=c["mode"], **s["opts"])]
        else:
            r = s["B"].relax(s["Xs"], s["Ps"], mode=c["mode"], **s["opts"])
        return {"X": s["X"], "counts": np.array([[x["iters"], x["n_t1"], x["n_stretch"],
                                                  x["status"]] for x in r]),
                "energy": np.array([x["energy"] for x in r]),
                "max_f": np.array([x["max_f"] for x in r])}
    if kind == "fit":
        # the outer cost is the mean squared distance to the target, minimum image
        theta = s["theta"]
        theta.grad = None
        X = equilibrium(theta, s["X"], s["T"], s["P"], which="lambda", mode="f64",
                        relax=dict(eta=1e-2, tol=1e-3, patience=10, max_iter=1000,
                                   t1_enable=True, l_min=5e-3),
                        grad=dict(method="adjoint", cg_tol=1e-12))
        d = X - s["Xt"]
        d = d - s["box"] * torch.floor(d / s["box"] + 0.5)
        ((d * d).sum() / (2 * X.shape[0])).backward()
        return {"X": X.detach(), "grad": theta.grad}
    if kind == "ep":
        return s["B"].param_grad(s["Xs"], s["Ps"], X_target=s["Xt"], method="ep",
                                 theta=c["theta"], beta=1e-2,
                                 ep_relax=dict(eta=3e-3, tol=0.0, max_iter=c["steps"]))[0]
    if c["how"] == "sens":
        out, w, _ = s["Ts"][0].param_sens(s["Xs"][0], s["Ps"][0], s["d"], s["b"][0],
                                          theta=c["theta"], cg_tol=1e-12, want_dX=True)
        return {"dC": out, "dX": w}
    method = "adjoint" if c["how"] == "adjoint" else "adjoint_minres"
    kw = dict(method=method, theta=c["theta"], cg_tol=1e-12)
    if s["B"] is None:
        return s["Ts"][0].param_grad(s["Xs"][0], s["Ps"][0], dC_dX=s["b"][0], **kw)[0]
    # one array over the tissues, as an optimiser of all parameters takes it
    return torch.cat(s["B"].param_grad(s["Xs"], s["Ps"], dC_dX=s["b"], **kw)[0])


# ---------------------------------------------------------------------- work
def work(case):
    """Bytes of the inputs and outputs of a pass, once each, and about the
    floating-point operations of its steps (an evaluation: 110 a vertex; a
    Hessian-vector product: 160)."""
    kind = case["kind"]
    if kind == "eval":
        nv = 2 * case["patch"] * case["rep"] ** 2
        w = 4 if case["mode"] == "f32" else 8
        # positions, forces, one 3-neighbour list, each tension once, P0
        return {"bytes": nv * (4 * w + 12 + 1.5 * w + (0.5 * w if case["hetero"] else 0)),
                "flops": 110.0 * nv}
    if kind == "relax":
        nv = 2 * sum(n for n, _ in _sizes(case))
        w = 4 if case["mode"] == "f32" else 8
        return {"bytes": nv * (4 * w + 12 + 2 * w), "flops": 110.0 * nv * case["steps"]}
    nv = 2 * case["cells"] * case.get("tissues", 1)
    if kind == "fit":  # about 300 descent steps and 100 CG steps
        return {"bytes": nv * 80, "flops": (300 * 110.0 + 100 * 160.0) * nv}
    if kind == "ep":
        return {"bytes": nv * 80, "flops": 110.0 * nv * 2 * case["steps"]}
    # CG steps grow with the linear size
    return {"bytes": nv * 80, "flops": 160.0 * nv * 30 * math.sqrt(case["cells"])}


# --------------------------------------------------------------------- exact
def _descend(m, X, P0, lam, steps, nudge=None, eta=3e-3):
    for _ in range(steps):
        F = m.force(X, P0, lam)
        if nudge is not None:
            F = F - nudge(X)
        X = X + eta * F
    return X, F


def _grad_of(m, X, theta, mu):
    """-(d2E/dX dtheta)^T mu."""
    if theta == "lambda":
        return -torch.func.jvp(lambda x: m.lengths(x)[0], (X,), (mu,))[1]
    return 2 * torch.func.jvp(lambda x: m.cell(x)[1], (X,), (mu,))[1]


def exact(case, seed):
    kind = case["kind"]
    if kind == "eval":
        t, X, P0, lam = _eval_inputs(case, seed)
        m, X, lam = _Model([t]), X.to(F64), lam.to(F64)
        P0 = P0.to(F64) if case["hetero"] else P0
        Ec, Ee = m.energy(X, P0, lam)
        F = m.force(X, P0, lam)
        return Ec.sum() + Ee.sum(), F, F.abs().max()
    if kind == "relax":
        if case["t1"] or case["steps"] * sum(n for n, _ in _sizes(case)) > 1 << 26:
            return None
        ts, X, P0, lam = _relax_inputs(case, seed)
        m, X, P0, lam = _Model(ts), X.to(F64), P0.to(F64), lam.to(F64)
        X, F = _descend(m, X, P0, lam, case["steps"])
        Ec, Ee = m.energy(X, P0, lam)
        E = [a.sum() + b.sum() for a, b in zip(_split(Ec, [t.n_cell for t in ts]),
                                               _split(Ee, [t.n_edge for t in ts]))]
        mf = [f.abs().max() for f in _split(F, [t.n_vert for t in ts])]
        return {"X": X, "counts": None, "energy": torch.stack(E), "max_f": torch.stack(mf)}
    if kind == "fit":
        s = prepare(case, seed)
        ts, m, X, P0, _, Xt, _ = _solve_inputs({"cells": case["cells"], "tissues": 1}, seed)
        lam, count = s["theta"].detach(), 0
        for k in range(1000):
            if float(m.lengths(X)[0].min()) < 6e-3:
                return None  # an exchange may follow
            F = m.force(X, P0, lam)
            count = count + 1 if float(F.abs().max()) < 1e-3 else 0
            if count >= 10:
                break
            X = X + 1e-2 * F
        d = X - Xt
        d = d - s["box"] * torch.floor(d / s["box"] + 0.5)
        mu = _cg(m, X, P0, lam, d / X.shape[0], 1)
        return {"X": X, "grad": _grad_of(m, X, "lambda", mu)}
    ts, m, X, P0, lam, Xt, d = _solve_inputs(case, seed)
    n_t, nv = len(ts), ts[0].n_vert
    ns = [t.n_edge if case["theta"] == "lambda" else t.n_cell for t in ts]
    if kind == "ep":
        def nudge(beta):
            def f(x):
                c = ((x - Xt) / nv).reshape(n_t, nv, 2)
                return beta * (c - c.mean(1, keepdim=True)).reshape(-1, 2)
            return f
        got = []
        for sgn in (1.0, -1.0):
            Y = _descend(m, X, P0, lam, case["steps"], nudge(sgn * 5e-3))[0]
            got.append(m.lengths(Y)[0] if case["theta"] == "lambda" else -2 * (m.cell(Y)[1] - P0))
        return _split((got[0] - got[1]) / 1e-2, ns)
    b = (X - Xt) / nv
    if case["how"] == "sens":
        zero_c, zero_e = torch.zeros_like(P0), torch.zeros_like(lam)
        rhs = m.pull(X, zero_c, zero_c, d) if case["theta"] == "lambda" else \
            -m.pull(X, zero_c, 2 * d, zero_e)
        w = _cg(m, X, P0, lam, rhs, 1)
        return {"dC": (b * w).sum(), "dX": w}
    return _grad_of(m, X, case["theta"], _cg(m, X, P0, lam, b, n_t))
