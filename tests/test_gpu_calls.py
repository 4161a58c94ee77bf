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
