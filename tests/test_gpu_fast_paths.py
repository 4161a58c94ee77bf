"""Kernel variants chosen by size, at the edges of their ranges."""
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


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
def test_tile_tables_follow_a_batched_relaxation(vtx, mode):
    """The tables of a batch are rebuilt in one launch, and only for tissues
    that made an exchange: afterwards every tissue's fused forces equal the
    two passes' (which read the rows and stars) bit for bit.  Sizes around a
    tile of 256 vertices, and a hexagonal tiling that makes no exchange."""
    V = vtx
    dt = V.pos_dtype(mode)
    ts = [g.random_tissue(n, seed=40 + n) for n in (20, 127, 128, 129, 257, 700)]
    ts.append(g.hex_lattice(6, 6, float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0))))))
    Ts = [V.Tissue.from_tissue(t) for t in ts]
    Xs = [_dev(t.X, dt) for t in ts]
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1)
    for _ in range(2):  # the second call starts from tables rebuilt by the first
        res = V.Batch(Ts).relax(Xs, [P] * len(Ts), mode=mode, eta=3e-3, tol=0.0, max_iter=150,
                                t1_enable=True, l_min=0.02)
        for T, X in zip(Ts, Xs):
            F = T.energy_forces(X, P, mode=mode)[1]
            F2, _ = T.vertex_forces(X, P, T.cell_coeffs(X, P, mode=mode), mode=mode)
            assert torch.equal(F, F2)
    assert res[-1]["n_t1"] == 0 and any(r["n_t1"] > 0 for r in res)


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("n_cell", [20, 32, 33, 64, 129, 255, 257, 513, 1000])
def test_one_workgroup_relaxation_matches_the_oracle(vtx, oracle, mode, n_cell):
    """Tissue.relax of a tissue that fits one workgroup (a wave for every 64
    vertices, at most eight; one cell per thread up to 512 cells, then two),
    with T1, at sizes around those steps.  In FP64 60 steps agree with the
    oracle to rounding (each step adds at most a few ulp of the box side);
    the reduced modes to 60 steps of their force rounding."""
    V = vtx
    t = g.random_tissue(n_cell, seed=300 + n_cell)
    p = g.uniform_params(t, P0=3.7, lam=0.1)
    T = V.Tissue.from_tissue(t)
    X = _dev(t.X, V.pos_dtype(mode))
    opts = dict(eta=3e-3, tol=0.0, max_iter=60, t1_enable=True, l_min=0.02)
    r = T.relax(X, V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.7, lam=0.1), mode=mode, **opts)
    m = oracle.Mesh.from_tissue(t)
    Xo = t.X.astype(np.float32).astype(np.float64) if mode == "f32" else t.X.copy()
    ro = oracle.relax(m, Xo, p, patience=1, **opts)
    assert r["iters"] == ro["iters"] == 60
    if mode != "f64":
        # an edge within rounding of the threshold may be handled a step apart
        same = np.array_equal(T.topology(), m.he)
        if not same:
            return
    assert np.array_equal(T.topology(), m.he)
    assert (r["n_t1"], r["n_stretch"]) == (ro["n_t1"], ro["n_stretch"])
    ulp = {"f64": 2.0 ** -52, "mixed": 2.0 ** -23 * 3e-3, "f32": 2.0 ** -23}[mode]
    err = np.abs(X.cpu().numpy() - Xo).max()
    assert err <= 60 * 16 * ulp * max(t.Lx, 20.0), err


@pytest.mark.parametrize("scale", [1e-60, 1e-3, 1.0, 1e60])
def test_fp64_lengths_over_the_range(vtx, oracle, scale):
    """Forces and energy of a tissue scaled over the exponent range of the
    FP64 lengths (areas up to scale^2, their squares up to scale^4)."""
    V = vtx
    t = g.random_tissue(100, seed=7)
    ts = g.Tissue(t.he, t.X * scale, t.Lx * scale, t.Ly * scale)
    p = g.uniform_params(ts, A0=scale ** 2, P0=3.7 * scale, lam=0.1 * scale,
                         KA=scale ** -2)
    T = V.Tissue.from_tissue(ts)
    P = V.Params(KA=scale ** -2, A0=scale ** 2, KP=1.0, P0=3.7 * scale, lam=0.1 * scale)
    E, F, _ = T.energy_forces(_dev(ts.X), P)
    Eo, Fo = oracle.energy_forces(oracle.Mesh.from_tissue(ts), ts.X, p)
    assert abs(E.item() / Eo - 1.0) < 1e-12
    assert np.abs(F.cpu().numpy() - Fo).max() / np.abs(Fo).max() < 1e-12


@pytest.mark.parametrize("method", ["adjoint", "adjoint_minres"])
@pytest.mark.parametrize("theta", ["lambda", "P0"])
@pytest.mark.parametrize("n_cell", [20, 32, 33, 129, 256, 257, 512, 513, 1000, 1024, 1025])
def test_one_workgroup_solve_matches_the_oracle(vtx, oracle, n_cell, theta, method):
    """Gradients of single FP64 tissues at the steps of the one-workgroup
    solve (a wave for every 64 vertices, at most eight; one cell per thread up
    to 512, then two; beyond 1024 cells the whole GPU), on random tilings
    (3- to 12-sided cells) under tensions that make H positive definite.
    Both solvers stop at a residual of 1e-12, so gradients agree to that
    times the condition number (below 1e5 here)."""
    V = vtx
    t = g.random_tissue(n_cell, seed=900 + n_cell)
    rng = np.random.default_rng(n_cell)
    p = g.uniform_params(t, KA=0.02, P0=0.5, lam=1.0)
    p.lam = rng.uniform(0.9, 1.1, t.n_edge)
    b = rng.normal(size=(t.n_vert, 2))
    T = V.Tissue.from_tissue(t)
    P = V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=_dev(p.lam))
    got, info = T.param_grad(_dev(t.X), P, dC_dX=_dev(b), theta=theta, method=method,
                             cg_tol=1e-12)
    ref, info_o = oracle.adjoint_grad(oracle.Mesh.from_tissue(t), t.X, p, b, theta=theta,
                                      tol=1e-12)
    assert info["status"] == V.CONVERGED and info_o["status"] == 0
    assert info["cg_rel_res"] <= 1e-12
    err = np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max()
    assert err < 1e-7, err
    # a batch of the tissue and a smaller one takes the same kernel
    if n_cell == 513:
        t2 = g.random_tissue(40, seed=5)
        T2 = V.Tissue.from_tissue(t2)
        P2 = V.Params(KA=0.02, P0=0.5, lam=1.0)
        outs, _ = V.Batch([T2, T]).param_grad([_dev(t2.X), _dev(t.X)], [P2, P],
                                              dC_dX=[_dev(np.ones((80, 2))), _dev(b)],
                                              theta=theta, method=method, cg_tol=1e-12)
        assert torch.equal(outs[1], got)
        assert float(outs[0].abs().max()) == 0.0  # a constant cost gradient has no zero-mean part


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("t1", [True, False])
@pytest.mark.parametrize("n_cell,chunk", [(1025, 0), (1500, 1), (2111, 17)])
def test_one_launch_step_equals_the_batched_loop(vtx, mode, t1, n_cell, chunk):
    """Tissue.relax beyond one workgroup takes one launch per iteration (three
    with a T1 pass, whatever the length of the captured chunk): the iterates,
    counts and topology are those of the batched loop bit for bit, at a fixed
    number of steps and at a tolerance with patience."""
    V = vtx
    dt = V.pos_dtype(mode)
    t = g.random_tissue(n_cell, seed=70 + n_cell)
    rng = np.random.default_rng(n_cell)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=_dev(rng.uniform(3.6, 3.9, t.n_cell), dt),
                 lam=_dev(rng.uniform(0.05, 0.15, t.n_edge), dt))
    for kw in (dict(tol=0.0, max_iter=101), dict(tol=0.8, max_iter=400, patience=7)):
        T1, T2 = V.Tissue.from_tissue(t), V.Tissue.from_tissue(t)
        X1, X2 = _dev(t.X, dt), _dev(t.X, dt)
        opts = dict(eta=3e-3, t1_enable=t1, l_min=0.02, **kw)
        r1 = T1.relax(X1, P, mode=mode, chunk=chunk, **opts)
        r2 = V.Batch([T2]).relax([X2], [P], mode=mode, block_threads=1024, **opts)[0]
        keys = ("iters", "n_t1", "n_stretch", "status", "max_f")
        assert [r1[k] for k in keys] == [r2[k] for k in keys]
        assert torch.equal(X1, X2) and np.array_equal(T1.topology(), T2.topology())
        assert not t1 or r1["n_t1"] > 0
        # the tables of the fused evaluation follow
        F = T1.energy_forces(X1, P, mode=mode)[1]
        assert torch.equal(F, T1.vertex_forces(X1, P, T1.cell_coeffs(X1, P, mode=mode),
                                               mode=mode)[0])


def _fan(n_petals):
    """A tiling with one cell of many sides: n_petals seeds on a circle around
    one, the rest at random outside."""
    L = 14.0
    rng = np.random.default_rng(n_petals)
    a = 2.0 * np.pi * (np.arange(n_petals) + 0.3) / n_petals
    ring = 7.0 + 2.0 * np.stack([np.cos(a), np.sin(a)], 1)
    out = rng.uniform(0.0, L, size=(400, 2))
    out = out[np.hypot(*(out - 7.0).T) > 2.6][:150]
    return g.periodic_voronoi(np.concatenate([[[7.0, 7.0]], ring, out]), L, L)


@pytest.mark.parametrize("mode", ["f64", "f32"])
@pytest.mark.parametrize("petals", [12, 13, 14, 15, 16, 22])
def test_t1_pass_around_long_rows(vtx, oracle, petals, mode):
    """T1 passes next to a cell of 12 to 22 sides: rows of up to 14 corners
    are evaluated and edited by 16 lanes, longer ones by one.  Topology and
    counts are the oracle's exactly."""
    V = vtx
    t = _fan(petals)
    sides = np.bincount(t.he[:, g.HE_FACE])
    assert sides.max() == petals
    p = g.uniform_params(t, P0=3.6, lam=0.1)
    X = _dev(t.X, V.pos_dtype(mode))
    Xo = X.cpu().numpy().astype(np.float64)
    T, m = V.Tissue.from_tissue(t), oracle.Mesh.from_tissue(t)
    for l_min in (0.05, 1.2 * 2.0 * np.pi / petals):  # the second takes the long cell's own sides
        got = T.t1(X, V.Params(P0=3.6, lam=0.1), l_min, mode=mode)
        ref = oracle.t1_pass(m, Xo, p, l_min, 2.0 * l_min)
        if mode == "f32":  # the oracle goes on from the stored positions
            Xo = X.cpu().numpy().astype(np.float64)
        assert got[0] > 0 and tuple(got) == tuple(ref)[:2]
        assert np.array_equal(T.topology(), m.he)
    F = T.energy_forces(X, V.Params(P0=3.6, lam=0.1), mode=mode)[1]
    Fo = oracle.energy_forces(m, Xo, p)[1]
    assert np.abs(F.cpu().numpy() - Fo).max() / np.abs(Fo).max() < (1e-10 if mode == "f64" else 1e-5)


@pytest.mark.parametrize("make,theta", [("random", "lambda"), ("random", "P0"), ("hex", "P0"),
                                        ("fan", "lambda")])
def test_one_launch_cg_matches_the_oracle(vtx, oracle, make, theta):
    """CG beyond one workgroup runs on the assembled rows of the Hessian, one
    launch per iteration: random tilings (3 to 12 sides), hexagons (no row
    longer than the least width) and a cell of 22 sides (a wider table), the
    last two after a smaller table was built for the same tissue.  Step counts
    agree with the oracle's to one (sums are added in another order) and
    gradients to the residual of 1e-12 times the condition number."""
    V = vtx
    rng = np.random.default_rng(12)
    if make == "random":
        t = g.random_tissue(1500, seed=31)
    elif make == "hex":
        t = g.hex_lattice(34, 34, float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0)))))
    else:
        one = _fan(22)
        seeds = np.concatenate([one.seeds + [14.0 * i, 14.0 * j] for i in range(3) for j in range(3)])
        t = g.periodic_voronoi(seeds, 42.0, 42.0)
        assert t.n_cell > 1024 and np.bincount(t.he[:, g.HE_FACE]).max() == 22
    p = g.uniform_params(t, KA=0.02, P0=0.5, lam=1.0)
    p.lam = rng.uniform(0.9, 1.1, t.n_edge)
    b = rng.normal(size=(t.n_vert, 2))
    T, m = V.Tissue.from_tissue(t), oracle.Mesh.from_tissue(t)
    P = V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=_dev(p.lam))
    got, info = T.param_grad(_dev(t.X), P, dC_dX=_dev(b), theta=theta, cg_tol=1e-12)
    ref, info_o = oracle.adjoint_grad(m, t.X, p, b, theta=theta, tol=1e-12)
    assert info["status"] == V.CONVERGED and info["cg_rel_res"] <= 1e-12
    assert abs(info["cg_iters"] - info_o["iters"]) <= 0.02 * info_o["iters"] + 1
    assert np.abs(got.cpu().numpy() - ref).max() / np.abs(ref).max() < 1e-7
    # the residual of the solution, through the separate product
    d = _dev(rng.normal(size=t.n_edge if theta == "lambda" else t.n_cell))
    _, w, _ = T.param_sens(_dev(t.X), P, d, _dev(b), theta=theta, cg_tol=1e-12, want_dX=True)
    Hw = oracle.hvp(m, t.X, p, w.cpu().numpy())
    Hg = T.hvp(_dev(t.X), P, w).cpu().numpy()
    assert np.abs(Hw - Hg).max() / np.abs(Hw).max() < 1e-11
    # stopping at the step limit and at a constant (zero-mean zero) right side
    _, i1 = T.param_grad(_dev(t.X), P, dC_dX=_dev(b), theta=theta, cg_tol=1e-12, cg_max_iter=5)
    assert (i1["cg_iters"], i1["status"]) == (5, V.CG_MAXITER)
    g0, i0 = T.param_grad(_dev(t.X), P, dC_dX=_dev(np.ones_like(b)), theta=theta, cg_tol=1e-12)
    assert (i0["cg_iters"], i0["status"]) == (0, V.CONVERGED) and float(g0.abs().max()) == 0.0
    # a state that is no minimum stops with the curvature status
    Pn = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=6.0, lam=-1.0)
    _, i2 = T.param_grad(_dev(t.X), Pn, dC_dX=_dev(b), theta=theta, cg_tol=1e-12)
    assert i2["status"] == V.CG_NEG_CURVATURE


@pytest.mark.parametrize("rows", [40, 96, 132])
def test_one_launch_cg_takes_any_vertex_numbering(vtx, rows):
    """A workgroup of the CG step keeps the columns that it reads of other
    workgroups in LDS, up to 1024: vertices numbered at random need 625 to 715
    of them at 64 vertices a workgroup (several per thread), up to 956 at 80
    and 1638 or more at 144, beyond the room there is.  The gradient is that of the tissue numbered in
    space; both solve to a residual of 1e-12."""
    V = vtx
    rng = np.random.default_rng(rows)
    t = g.hex_lattice(rows, rows, float(np.sqrt(2.0 / (3.0 * np.sqrt(3.0)))))
    X = t.X + 0.02 * rng.normal(size=t.X.shape)
    b, lam = rng.normal(size=X.shape), rng.uniform(0.9, 1.1, t.n_edge)
    to = rng.permutation(t.n_vert)
    he = t.he.copy()
    for col in (g.HE_SRC, g.HE_TGT):
        he[:, col] = to[he[:, col]]
    back = np.argsort(to)
    P = V.Params(KA=0.02, A0=1.0, KP=1.0, P0=0.5, lam=_dev(lam))
    out = []
    for tis, x, rhs in ((t, X, b), (g.Tissue(he, X[back], t.Lx, t.Ly), X[back], b[back])):
        T = V.Tissue.from_tissue(tis)
        got, info = T.param_grad(_dev(x), P, dC_dX=_dev(rhs), theta="lambda", cg_tol=1e-12)
        assert info["status"] == V.CONVERGED
        out.append((got.cpu().numpy(), info["cg_iters"]))
    assert abs(out[0][1] - out[1][1]) <= 0.02 * out[0][1] + 1
    assert np.abs(out[0][0] - out[1][0]).max() / np.abs(out[0][0]).max() < 1e-9


@pytest.mark.parametrize("steps", [1, 6, 39, 40, 61, 253, 292])
@pytest.mark.parametrize("path", ["t1", "plain", "nudged"])
def test_relaxation_steps_queued_before_a_status_read(vtx, path, steps):
    """Without a `chunk` the loop queues as many steps as are left (graphs of
    60, the last third of one launched directly, a status read after 252 at
    most); the result is that of graphs of 7 with a read after each, bit for
    bit, and T1 iterations, which take more launches, are all made."""
    V = vtx
    t = g.random_tissue(1400, seed=3)
    rng = np.random.default_rng(steps)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=3.75, lam=_dev(rng.uniform(0.05, 0.15, t.n_edge)))
    kw = dict(eta=0.01, tol=0.0, patience=1, max_iter=steps)
    if path == "t1":
        kw.update(t1_enable=True, l_min=0.05, l_new=0.06)
    if path == "nudged":
        kw.update(beta=0.01, X_target=_dev(t.X + 0.01 * rng.normal(size=t.X.shape)))
    out = []
    for chunk in (0, 7):
        T, X = V.Tissue.from_tissue(t), _dev(t.X)
        info = T.relax(X, P, chunk=chunk, **kw)
        out.append((X.cpu().numpy(), info["iters"], info["n_t1"], info["status"]))
    assert out[0][1] == steps and out[0][1:] == out[1][1:]
    assert np.array_equal(out[0][0], out[1][0])


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("cells,threads", [((1025, 2048), 512), ((2049, 1100), 512),
                                           ((4096, 1300), 1024), ((4097, 1300), 1024)])
def test_batched_positions_in_lds_equal_the_grid(vtx, mode, cells, threads):
    """The general batched kernel keeps the positions of up to eight vertices
    per thread in LDS and those of larger tissues in global memory: iterates,
    counts and topology of both, through exchanges that move rows and change
    images, are those of Tissue.relax bit for bit."""
    V = vtx
    dt = V.pos_dtype(mode)
    ts = [g.random_tissue(n, seed=90 + n) for n in cells]
    rng = np.random.default_rng(cells[0])
    Ps = [V.Params(KA=1.0, A0=_dev(rng.uniform(0.9, 1.1, t.n_cell), dt), KP=1.0, P0=3.75,
                   lam=_dev(rng.uniform(0.05, 0.15, t.n_edge), dt)) for t in ts]
    opts = dict(eta=3e-3, t1_enable=True, l_min=0.03, tol=0.0, max_iter=120)
    A, B = ([V.Tissue.from_tissue(t) for t in ts] for _ in range(2))
    XA, XB = ([_dev(t.X, dt) for t in ts] for _ in range(2))
    got = V.Batch(A).relax(XA, Ps, mode=mode, block_threads=threads, **opts)
    for i, t in enumerate(ts):
        ref = B[i].relax(XB[i], Ps[i], mode=mode, **opts)
        keys = ("iters", "n_t1", "n_stretch", "status", "max_f")
        assert [got[i][k] for k in keys] == [ref[k] for k in keys] and ref["n_t1"] > 50
        assert torch.equal(XA[i], XB[i]) and np.array_equal(A[i].topology(), B[i].topology())


@pytest.mark.parametrize("mode", ["f32", "mixed", "f64"])
@pytest.mark.parametrize("window", [1, 300, 400, 512])
def test_fused_evaluation_lists_of_any_length(vtx, mode, window):
    """A tile reads the first 192 cells and halo vertices and 1024 corner
    references of its lists ahead of their lengths.  Vertices numbered at
    random within a window give lists of 118 to 171 cells (1), to 316 cells and
    515 halo vertices (300), always beyond 192 and 1024 (512), and some tiles
    that fit no list (400): forces and max |F| are those of the two passes, bit
    for bit, with per-cell and per-edge parameters."""
    V = vtx
    dt = V.pos_dtype(mode)
    t = g.random_tissue(1500, seed=8)
    rng = np.random.default_rng(window)
    to = np.arange(t.n_vert)
    for a in range(0, t.n_vert, window):
        to[a:a + window] = a + rng.permutation(min(window, t.n_vert - a))
    he = t.he.copy()
    for col in (g.HE_SRC, g.HE_TGT):
        he[:, col] = to[he[:, col]]
    t = g.Tissue(he, t.X[np.argsort(to)], t.Lx, t.Ly)
    T, X = V.Tissue.from_tissue(t), _dev(t.X, dt)
    assert (T.tile_stats()["global_tiles"] > 0) == (window == 400)
    P = V.Params(KA=1.0, A0=1.0, KP=1.0, P0=_dev(rng.uniform(3.6, 3.9, t.n_cell), dt),
                 lam=_dev(rng.uniform(0.05, 0.15, t.n_edge), dt))
    _, F, maxf = T.energy_forces(X, P, mode=mode, want_maxf=True)
    F2, maxf2 = T.vertex_forces(X, P, T.cell_coeffs(X, P, mode=mode), mode=mode, want_maxf=True)
    assert torch.equal(F, F2) and float(maxf) == float(maxf2)
