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
