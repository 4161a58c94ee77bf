"""What the calls promise besides their values on one stream: results that are
complete when a synchronising call returns, input that is not finite, memory,
threads, and both sides of every choice of a path by size."""
import numpy as np
import pytest
import torch

from paper_2604_06896_amd import tissue_gen as g

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="session")
def vtx():
    from paper_2604_06896_amd import vtx as V
    V.lib()
    return V


def _dev(a, dtype=torch.float64):
    return torch.as_tensor(np.asarray(a), dtype=dtype, device="cuda")


@pytest.mark.parametrize("n_cell", [100, 1000, 1500])
@pytest.mark.parametrize("schedule", ["relax", "grid", "persistent", "t1"])
def test_tables_are_complete_when_a_call_with_exchanges_returns(vtx, n_cell, schedule):
    """A call that made exchanges on one stream is followed at once by an
    evaluation on another, which reads the tile tables: the forces are those
    of the two passes (which read the rows and stars) bit for bit.  The calls
    synchronise their stream, the rebuild of the tables with it."""
    V = vtx
    t = g.random_tissue(n_cell, seed=n_cell)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1)
    T, X = V.Tissue.from_tissue(t), _dev(t.X)
    A, B = torch.cuda.Stream(), torch.cuda.Stream()
    E, F = torch.empty((), dtype=torch.float64, device="cuda"), torch.empty_like(X)
    cp, _ = P.to_c(X.dtype, X.device)
    batch = V.Batch([T])  # (kept: its end would synchronise the device)
    torch.cuda.synchronize()
    total = 0
    for _ in range(3):
        with torch.cuda.stream(A):
            kw = dict(eta=3e-3, tol=0.0, max_iter=40, t1_enable=True, l_min=0.05)
            if schedule == "relax":
                n_t1 = T.relax(X, P, **kw)["n_t1"]
            elif schedule == "t1":
                n_t1 = T.t1(X, P, 0.1)[0]
            else:
                how = V.SCHED_GRID if schedule == "grid" else V.SCHED_PERSISTENT
                n_t1 = batch.relax([X], [P], mode="f64", schedule=how, **kw)[0]["n_t1"]
        with torch.cuda.stream(B):
            T.energy_forces_into(X, cp, E, F, mode="f64")
            F2 = T.vertex_forces(X, P, T.cell_coeffs(X, P))[0]
        torch.cuda.synchronize()
        assert torch.equal(F, F2)
        total += n_t1
        if schedule == "t1":  # shorten edges for the next pass
            T.relax(X, P, eta=3e-3, tol=0.0, max_iter=20)
    assert total > 0


def _stiff(t, seed=0):
    """Parameters under which H is positive definite on any tiling."""
    rng = np.random.default_rng(seed)
    return dict(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=rng.uniform(0.9, 1.1, t.n_edge))


@pytest.mark.parametrize("bad", [np.nan, np.inf, 1e200])
@pytest.mark.parametrize("method", ["adjoint", "adjoint_minres"])
@pytest.mark.parametrize("mode,n_cell", [("f64", 1000), ("f64", 1025), ("mixed", 200)])
def test_a_right_side_that_is_not_finite_is_not_solved(vtx, mode, n_cell, method, bad):
    """One NaN or infinity in dC/dX, or a norm whose square overflows: no solver
    reports convergence (one workgroup, one launch per step, the general
    loops, batches of each form).  A scale that stays in range scales the
    gradient."""
    V = vtx
    t = g.random_tissue(n_cell, seed=5)
    kw = _stiff(t)
    lam = kw.pop("lam")
    P = V.Params(lam=_dev(lam), **kw)
    T, X = V.Tissue.from_tissue(t), _dev(t.X)
    rng = np.random.default_rng(1)
    unit = rng.normal(size=(t.n_vert, 2))
    b = unit * bad if bad == 1e200 else unit.copy()
    b[7, 1] *= bad if bad != 1e200 else 1.0
    opts = dict(mode=mode, method=method, cg_tol=1e-10)
    got = [T.param_grad(X, P, dC_dX=_dev(b), **opts)]
    for threads in (0, 1024) + ((-2,) if mode == "f64" and method == "adjoint" else ()):
        out, info = V.Batch([T]).param_grad([X], [P], dC_dX=[_dev(b)], block_threads=threads, **opts)
        got.append((out[0], info[0]))
    for grad, info in got:
        assert (info["status"], info["cg_iters"]) == (V.CG_MAXITER, 0)
        assert np.isnan(info["cg_rel_res"]) and float(grad.abs().max()) == 0.0
    if bad == 1e200 and mode == "f64":
        ref, info = T.param_grad(X, P, dC_dX=_dev(unit), **opts)
        for scale in (1e140, 1e-140):
            big, i2 = T.param_grad(X, P, dC_dX=_dev(unit * scale), **opts)
            assert info["status"] == i2["status"] == V.CONVERGED
            assert float((big / scale - ref).abs().max() / ref.abs().max()) < 1e-7


def _flower(n_cell, sides, seed=0):
    """About n_cell random cells around one of `sides` sides."""
    L, rng = np.sqrt(n_cell), np.random.default_rng([n_cell, sides, seed])
    R = max(1.2, 0.3 * sides / (2.0 * np.pi))
    a = 2.0 * np.pi * (np.arange(sides) + 0.3) / sides
    out = rng.uniform(0.0, L, size=(n_cell, 2))
    out = out[np.hypot(*(out - L / 2).T) > R + 0.6]
    ring = L / 2 + R * np.stack([np.cos(a), np.sin(a)], 1)
    t = g.periodic_voronoi(np.concatenate([[[L / 2, L / 2]], ring, out]), L, L)
    assert np.bincount(t.he[:, g.HE_FACE]).max() == sides
    return t


@pytest.mark.parametrize("n_cell,sides", [(3000, 100), (6000, 118), (6000, 140), (9000, 100)])
def test_cg_memory_with_a_cell_of_many_sides(vtx, n_cell, sides):
    """The rows of the one-launch CG are as wide as the largest cell for every
    vertex, 144 bytes a vertex and slot: beyond 1.5 million slots the solve
    keeps the loop without them.  The memory a solve leaves held stays within
    that (plus a megabyte of lists and rounding of four allocations to 2 MiB),
    and its solution solves the system as the separate product has it."""
    V = vtx
    t = _flower(n_cell, sides)
    kw = _stiff(t)
    P = V.Params(lam=_dev(kw.pop("lam")), **kw)
    T, X = V.Tissue.from_tissue(t), _dev(t.X)
    rng = np.random.default_rng(3)
    b = _dev(rng.normal(size=t.X.shape))
    T.hvp(X, P, b)  # (what the first calls of a process allocate)
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    d = _dev(rng.normal(size=t.n_edge))
    _, w, info = T.param_sens(X, P, d, b, cg_tol=1e-10, want_dX=True)
    held = free - torch.cuda.mem_get_info()[0]
    slots = (sides - 2) * t.n_vert
    assert held <= (144 * 1.02 * slots if slots <= 1500000 else 0) + 12e6, held
    assert info["status"] == V.CONVERGED
    # H w = -(d2E/dX dlambda) d, by the difference of the forces along d: F is
    # linear in lambda, so the difference is exact up to rounding
    F0 = T.energy_forces(X, P)[1]
    F1 = T.energy_forces(X, V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=P.lam + d))[1]
    rhs = F1 - F0
    res = T.hvp(X, P, w) - (rhs - rhs.mean(0))
    assert float(res.norm() / rhs.norm()) < 1e-8


def test_calls_from_several_threads(vtx):
    """Four threads, each with its own stream and tissues, relax and solve
    tissues of different sizes at the same time: kernels of the same name with
    different amounts of LDS.  Every result is that of the same calls made
    alone."""
    import threading
    V = vtx
    sizes = (60, 300, 700, 1000)

    def work(n, rounds):
        t = g.random_tissue(n, seed=n)
        t2 = g.random_tissue(n + 1100, seed=n)
        kw = _stiff(t)
        P = V.Params(lam=_dev(kw.pop("lam")), **kw)
        P2 = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1)
        b = _dev(np.random.default_rng(n).normal(size=t.X.shape))
        T, T2 = V.Tissue.from_tissue(t), V.Tissue.from_tissue(t2)
        B2 = V.Batch([T2])
        out = []
        for _ in range(rounds):
            X, X2 = _dev(t.X), _dev(t2.X)
            T.relax(X, P2, eta=3e-3, tol=0.0, max_iter=15)
            B2.relax([X2], [P2], mode="f64", eta=3e-3, tol=0.0, max_iter=15)
            grad = T.param_grad(X, P, dC_dX=b, cg_tol=1e-3)[0]
            out.append((X, X2, grad))
        torch.cuda.current_stream().synchronize()
        return out

    ref = {n: work(n, 1)[0] for n in sizes}
    got, errors = {}, []

    def run(n):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                got[n] = work(n, 25)
        except Exception as e:  # reported by the test's own thread
            errors.append((n, repr(e)))

    threads = [threading.Thread(target=run, args=(n,)) for n in sizes]
    torch.cuda.synchronize()
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    torch.cuda.synchronize()
    assert not errors, errors
    for n in sizes:
        for r in got[n]:
            assert all(torch.equal(a, c) for a, c in zip(r, ref[n]))


def _hex(nx, ny, amp, seed=0):
    """A hexagonal tiling of nx x ny cells of area 1, its vertices displaced."""
    t = g.hex_lattice(nx, ny, float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0)))))
    rng = np.random.default_rng([nx, ny, seed])
    return g.Tissue(t.he, t.X + amp * rng.normal(size=t.X.shape), t.Lx, t.Ly)


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("nx,ny,t1", [(130, 130, True), (130, 130, False), (220, 222, True),
                                      (222, 222, True), (256, 256, False), (256, 258, False)])
def test_relaxation_on_both_sides_of_the_routes(vtx, mode, nx, ny, t1):
    """Tissue.relax around the largest tissue of the one-launch step (98304
    vertices with T1, 131072 without) and just above 32768 vertices, where a
    thread adds up more than two of its blocks' maxima: iterates, counts and
    topology are those of the batched loop bit for bit.  The first T1 pass of
    the larger ones sorts more candidates (5600) than fit in LDS (4096)."""
    V = vtx
    dt = V.pos_dtype(mode)
    t = _hex(nx, ny, 0.15)
    rng = np.random.default_rng(2)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=_dev(rng.uniform(3.6, 3.9, t.n_cell), dt),
                 lam=_dev(rng.uniform(0.05, 0.15, t.n_edge), dt))
    A, B = V.Tissue.from_tissue(t), V.Tissue.from_tissue(t)
    XA, XB = _dev(t.X, dt), _dev(t.X, dt)
    opts = dict(eta=3e-3, tol=0.0, max_iter=9, t1_enable=t1, l_min=0.3, l_new=0.35)
    ra = A.relax(XA, P, mode=mode, **opts)
    rb = V.Batch([B]).relax([XB], [P], mode=mode, block_threads=1024, **opts)[0]
    keys = ("iters", "n_t1", "n_stretch", "status", "max_f")
    assert [ra[k] for k in keys] == [rb[k] for k in keys]
    assert torch.equal(XA, XB) and np.array_equal(A.topology(), B.topology())
    if t1:
        first = V.Tissue.from_tissue(t).edge_lengths(_dev(t.X, dt), mode=mode) < 0.3
        assert ra["n_t1"] > 50 and (int(first.sum()) > 4096 or nx == 130)


@pytest.mark.parametrize("nx,ny", [(160, 126), (180, 180), (182, 182)])
def test_cg_on_both_sides_of_the_route(vtx, nx, ny):
    """FP64 CG with more than 144 vertices a workgroup, at its most (256; 64800
    vertices) and beyond the one-launch step (66248): the solution solves the
    system as the separate product has it."""
    V = vtx
    t = _hex(nx, ny, 0.02)
    kw = _stiff(t)
    P = V.Params(lam=_dev(kw.pop("lam")), **kw)
    T, X = V.Tissue.from_tissue(t), _dev(t.X)
    rng = np.random.default_rng(4)
    d, b = _dev(rng.normal(size=t.n_edge)), _dev(rng.normal(size=t.X.shape))
    dC, w, info = T.param_sens(X, P, d, b, cg_tol=1e-9, want_dX=True)
    assert info["status"] == V.CONVERGED and info["cg_rel_res"] <= 1e-9
    F0 = T.energy_forces(X, P)[1]
    F1 = T.energy_forces(X, V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=P.lam + d))[1]
    rhs = (F1 - F0) - (F1 - F0).mean(0)  # -(d2E/dX dlambda) d, exact up to rounding
    assert float((T.hvp(X, P, w) - rhs).norm() / rhs.norm()) < 1e-8
    assert abs(float(dC) - float((b * w).sum())) <= 1e-12 * float((b * w).abs().sum())


@pytest.mark.parametrize("rest", [0.0, 1e-9])
@pytest.mark.parametrize("n", [30, 34])
def test_cg_where_one_step_cuts_the_residual_sharply(vtx, oracle, n, rest):
    """On a perfect hexagonal tiling an eigenvector of H is solved for in one
    step, which cuts the residual to rounding, or to the 1e-9 of it that is
    spread over all others; the one-launch step (34 x 34 cells) has the next
    squared residual from a difference that cancels there.  The number of
    steps is the oracle's within a tenth, the gradient its to the tolerance
    times the condition number (below 1e4 here)."""
    V = vtx
    t = _hex(n, n, 0.0)
    m = oracle.Mesh.from_tissue(t)
    p = g.uniform_params(t, KA=0.02, P0=0.5, lam=1.0)
    # plane waves of one wave vector on the two vertices of a unit cell span
    # an invariant space: eight real dimensions
    k = 2.0 * np.pi * np.array([2.0 / t.Lx, 0.0])
    wave = [np.cos(t.X @ k), np.sin(t.X @ k)]
    cols = []
    # a vertex's sublattice: whether its vertical edge points up
    dy = (t.X[t.he[:, g.HE_TGT], 1] + t.he[:, g.HE_OY] * t.Ly - t.X[t.he[:, g.HE_SRC], 1])
    even = np.zeros(t.n_vert, bool)
    even[t.he[dy > 0.9 * dy.max(), g.HE_SRC]] = True
    assert even.sum() == t.n_cell
    for sub in (even, ~even):
        for w in wave:
            for comp in range(2):
                v = np.zeros_like(t.X)
                v[sub, comp] = w[sub]
                cols.append(v.ravel())
    Q, _ = np.linalg.qr(np.array(cols).T)
    HQ = np.stack([oracle.hvp(m, t.X, p, q.reshape(-1, 2)).ravel() for q in Q.T], 1)
    assert np.abs(HQ - Q @ (Q.T @ HQ)).max() < 1e-9  # invariant
    lam, U = np.linalg.eigh(Q.T @ HQ)
    b = (Q @ U[:, -1]).reshape(-1, 2)
    rng = np.random.default_rng(n)
    b = b / np.linalg.norm(b)
    noise = rng.normal(size=b.shape)
    b = b + rest * noise / np.linalg.norm(noise)
    T, P = V.Tissue.from_tissue(t), V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=1.0)
    ref, io = oracle.adjoint_grad(m, t.X, p, b, theta="lambda", tol=1e-13)
    got, info = T.param_grad(_dev(t.X), P, dC_dX=_dev(b), theta="lambda", cg_tol=1e-13)
    assert info["status"] == V.CONVERGED and io["status"] == 0
    assert abs(info["cg_iters"] - io["iters"]) <= 0.1 * io["iters"] + 1, (info, io)
    assert np.abs(got.cpu().numpy() - ref).max() < 1e-9 * np.abs(ref).max()


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("n_cell", [20, 32, 33, 64, 129, 255, 257, 513, 1000, 1024])
def test_one_workgroup_relaxation_in_every_mode(vtx, oracle, mode, n_cell):
    """Tissue.relax in one workgroup, in the reduced modes as well, with
    exchanges: one step has the oracle's topology and counts from the same
    stored positions (exchanges are decided in FP64 in every mode), and 80
    steps have the iterates, counts and topology of the general batched kernel
    (1024 threads) bit for bit, on a mesh whose forces are the oracle's."""
    V = vtx
    dt = V.pos_dtype(mode)
    t = g.random_tissue(n_cell, seed=600 + n_cell)
    p = g.uniform_params(t, P0=3.7, lam=0.1)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1)
    kw = dict(eta=3e-3, tol=0.0, t1_enable=True, l_min=0.05)
    T, X = V.Tissue.from_tissue(t), _dev(t.X, dt)
    m, Xo = oracle.Mesh.from_tissue(t), X.double().cpu().numpy()
    r, ro = T.relax(X, P, mode=mode, max_iter=1, **kw), oracle.relax(m, Xo, p, max_iter=1, **kw)
    assert (r["n_t1"], r["n_stretch"]) == (ro["n_t1"], ro["n_stretch"]) and r["n_stretch"] > 0
    assert np.array_equal(T.topology(), m.he)
    T2, X2 = V.Tissue.from_tissue(t), _dev(t.X, dt)
    T2.relax(X2, P, mode=mode, max_iter=1, **kw)
    ra = T.relax(X, P, mode=mode, max_iter=80, **kw)
    rb = V.Batch([T2]).relax([X2], [P], mode=mode, block_threads=1024, max_iter=80, **kw)[0]
    keys = ("iters", "n_t1", "n_stretch", "status", "max_f")
    assert [ra[k] for k in keys] == [rb[k] for k in keys]
    assert torch.equal(X, X2) and np.array_equal(T.topology(), T2.topology())
    F = T.energy_forces(X, P, mode=mode)[1].double().cpu().numpy()
    m.he[:] = T.topology()
    Fo = oracle.energy_forces(m, X.double().cpu().numpy(), p)[1]
    assert np.abs(F - Fo).max() / np.abs(Fo).max() < (1e-10 if mode == "f64" else 1e-5)
    assert V.Tissue.from_tissue(g.Tissue(m.he, Xo, t.Lx, t.Ly)).n_edge == t.n_edge  # a valid table


def _routes(V, t, mode="f64"):
    """Calls that relax tissue t, by name: each takes (X, params, options)."""
    T = V.Tissue.from_tissue(t)
    B = V.Batch([T])

    def batch(threads):
        return lambda X, P, **kw: B.relax([X], [P], mode=mode, block_threads=threads, **kw)[0]
    return T, {"single": lambda X, P, **kw: T.relax(X, P, mode=mode, **kw),
               "batch0": batch(0), "batch256": batch(256), "batch1024": batch(1024)}


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("n_cell", [300, 1000, 1100, 4200])
@pytest.mark.parametrize("t1", [False, True])
def test_forces_that_are_not_finite_end_every_loop(vtx, mode, n_cell, t1):
    """A step of 1e30, and a NaN in the positions: every loop (one workgroup
    from LDS, one launch per step, the general batched kernel with positions in
    LDS and in global memory) ends with VTX_E_NONFINITE at the positions whose
    forces are not finite, the same in all; the tissue is usable afterwards."""
    V = vtx
    dt = V.pos_dtype(mode)
    t = g.random_tissue(n_cell, seed=n_cell)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1)
    T, routes = _routes(V, t, mode)
    for bad in ("step", "nan"):
        X0 = t.X.copy()
        if bad == "nan":
            X0[n_cell // 2, 1] = np.nan
        ends = []
        for name, relax in routes.items():
            X = _dev(X0, dt)
            with pytest.raises(V.VtxError) as err:
                relax(X, P, eta=1e30 if bad == "step" else 1e-3, tol=0.0, max_iter=500,
                      t1_enable=t1, l_min=0.001)
            assert err.value.code == V.E_NONFINITE, name
            ends.append(X.cpu().numpy())
            T.set_topology(t.he)
        assert all(np.array_equal(ends[0], e, equal_nan=True) for e in ends)
        if bad == "nan" and not t1:  # (a T1 pass comes before the forces)
            assert np.array_equal(ends[0], _dev(X0, dt).cpu().numpy(), equal_nan=True)
    out = []
    for relax in routes.values():
        X = _dev(t.X, dt)
        relax(X, P, eta=1e-3, tol=0.0, max_iter=20)
        out.append(X)
    assert all(torch.equal(out[0], x) for x in out)


def _crowd(nx, ny):
    """A hexagonal tiling with short edges, no two near each other and all
    numbered before the rest, each of whose stretches shortens the four edges
    at its ends: (tissue, l_min, l_new, edges that wait for their turn)."""
    t = g.hex_lattice(nx, ny, float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0)))))
    side = float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0))))
    he = t.he
    assert np.array_equal(he[0::2, g.HE_TWIN], np.arange(1, len(he), 2))
    box = np.array([t.Lx, t.Ly])
    src, tgt = he[0::2, g.HE_SRC], he[0::2, g.HE_TGT]
    vec = t.X[tgt] + he[0::2, g.HE_OX:g.HE_OY + 1] * box - t.X[src]
    near = [set() for _ in range(t.n_vert)]
    for a, b in zip(src, tgt):
        near[a].add(b)
        near[b].add(a)
    X, used, chosen = t.X.copy(), set(), []
    for e in range(t.n_edge):
        a, b = src[e], tgt[e]
        zone = near[a] | near[b]
        if zone & used:
            continue
        used |= zone
        chosen.append(e)
        X[a] += 0.35 * vec[e]
        X[b] -= 0.35 * vec[e]
    order = np.array(chosen + [e for e in range(t.n_edge) if e not in set(chosen)])
    new = np.empty(t.n_edge, np.int64)
    new[order] = np.arange(t.n_edge)
    out = he.copy()
    for col in (g.HE_PREV, g.HE_NEXT, g.HE_TWIN):
        out[:, col] = 2 * new[he[:, col] // 2] + he[:, col] % 2
    out = out.reshape(-1, 2, 8)[order].reshape(-1, 8)
    return (g.Tissue(np.ascontiguousarray(out, np.int32), X, t.Lx, t.Ly), 0.95 * side, 2.0 * side,
            4 * len(chosen))


@pytest.mark.parametrize("mode", ["f32", "f64"])
@pytest.mark.parametrize("nx,ny", [(20, 20), (36, 32), (66, 66)])
def test_a_t1_pass_with_too_many_edges_waiting(vtx, oracle, mode, nx, ny):
    """More than 256 edges that became short wait for their turn in one T1 pass:
    VTX_E_CAPACITY from every loop and from the pass alone, and the tissue is
    as good as new after set_topology."""
    V = vtx
    dt = V.pos_dtype(mode)
    t, l_min, l_new, waiting = _crowd(nx, ny)
    assert waiting > 256
    # each short edge is stretched, not exchanged, and its four neighbours end short
    kw = dict(KA=1e-3, A0=1.0, KP=1e-3, P0=3.7, lam=1.0)
    m, Xo = oracle.Mesh.from_tissue(t), t.X.copy()
    before = oracle.edge_lengths(m, Xo) < l_min
    assert before.sum() == waiting // 4 and before[:waiting // 4].all()
    d = oracle.edge_lengths(m, Xo)
    src, tgt = t.he[0::2, g.HE_SRC], t.he[0::2, g.HE_TGT]
    vec = t.X[tgt] + t.he[0::2, g.HE_OX:g.HE_OY + 1] * np.array([t.Lx, t.Ly]) - t.X[src]
    for e in range(waiting // 4):
        Xo[src[e]] -= 0.5 * (l_new - d[e]) * vec[e] / d[e]
        Xo[tgt[e]] += 0.5 * (l_new - d[e]) * vec[e] / d[e]
    assert (oracle.edge_lengths(m, Xo) < l_min).sum() == waiting
    P = V.Params(**kw)
    T, routes = _routes(V, t, mode)
    routes["pass"] = lambda X, P, l_min, l_new, **_: T.t1(X, P, l_min, l_new, mode=mode)
    for name, relax in routes.items():
        with pytest.raises(V.VtxError) as err:
            relax(_dev(t.X, dt), P, eta=1e-6, tol=0.0, max_iter=3, t1_enable=True, l_min=l_min,
                  l_new=l_new)
        assert err.value.code == V.E_CAPACITY, name
        T.set_topology(t.he)
    out = []
    fresh = V.Tissue.from_tissue(t)
    for relax in [lambda X, P, **o: fresh.relax(X, P, mode=mode, **o)] + \
            [r for n, r in routes.items() if n != "pass"]:
        X = _dev(t.X, dt)
        relax(X, P, eta=1e-3, tol=0.0, max_iter=10, t1_enable=True, l_min=0.2 * l_min)
        out.append(X)
    assert all(torch.equal(out[0], x) for x in out)
