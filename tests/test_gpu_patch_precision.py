"""The path of a 3-D handle's FP32 cycle depends on the precision of the call, not on the one the handle was created
with: a handle created FP64 and switched gives the same bits as one created for the FP32 cycle."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


def _cube(n, item=0):
    X, T, _ = W.kuhn_cube_mesh(n, item=item)
    return X, T, np.exp(0.5 * np.random.default_rng(n).standard_normal(len(T)))


@pytest.mark.parametrize("n", [20, 31])
def test_single_mesh(n):
    mesh = _cube(n)
    created, switched = A.Solver(*mesh, precision=A.PREC_MIXED), A.Solver(*mesh)
    assert switched.info()["J"] > switched.info()["lc"]
    f = torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, created.n)).cuda()
    want = created.apply_preconditioner(f, A.PREC_MIXED)
    u, it, _ = created.solve_device(f, 1e-8)
    assert torch.equal(switched.apply_preconditioner(f, A.PREC_MIXED), want)
    z64 = switched.apply_preconditioner(f, A.PREC_FP64)
    for _ in range(2):
        switched.set_precision(A.PREC_MIXED)
        v, jt, _ = switched.solve_device(f, 1e-8)
        assert jt == it and torch.equal(u, v)
        switched.set_precision(A.PREC_FP64)
        switched.solve_device(f, 1e-8)
    assert torch.equal(switched.apply_preconditioner(f, A.PREC_FP64), z64)
    assert float((z64 - want).abs().max()) <= 1e-5 * float(z64.abs().max())


@pytest.mark.parametrize("nr", [1, 4])
def test_batch(nr):
    meshes = [_cube(n, n) for n in (6, 14, 20)]
    created, switched = A.BatchSolver(meshes, precision=A.PREC_MIXED), A.BatchSolver(meshes)
    f = torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, created.n_total * nr)).cuda()
    u, it, _ = created.solve(f, nr, 1e-8)
    w, _, _ = switched.solve(f, nr, 1e-8)
    for _ in range(2):
        switched.set_precision(A.PREC_MIXED)
        v, jt, _ = switched.solve(f, nr, 1e-8)
        assert (jt == it).all() and torch.equal(u, v)
        switched.set_precision(A.PREC_FP64)
        assert torch.equal(switched.solve(f, nr, 1e-8)[0], w)
