"""Overlapped patches (csrc/patch.hpp) against the oracle at the sizes where they can go wrong: no smoothed
auxiliary level, one patch, a last patch with few rows, a row longer than the entries kept in registers, matrix
values as codes (constant coefficient) and as values, and a change from one to the other on a live handle.

Bars as in the other parity tests: B_co element-wise within 1e-12 (FP64) and 1e-5 (FP32 V-cycle) of the oracle's.
"""
import numpy as np
import pytest

import workloads as W
from oracle.hierarchy import Hierarchy

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


def _rel_inf(a, b):
    return float(np.abs(a - b).max() / np.abs(b).max())


def _wheel(spokes=24, rings=14):
    """Rings of triangles around a centre of `spokes` neighbours (its matrix row has that many entries)."""
    t = 2 * np.pi * np.arange(spokes) / spokes
    p = [np.array([[0.5, 0.5]])]
    for k in range(1, rings + 1):
        r = 0.5 * k / rings
        p.append(np.stack([0.5 + r * np.cos(t + 0.1 * k), 0.5 + r * np.sin(t + 0.1 * k)], 1))
    i = np.arange(spokes)
    j = (i + 1) % spokes
    e = [np.stack([np.zeros(spokes, int), 1 + i, 1 + j], 1)]
    for k in range(rings - 1):
        a, b = 1 + k * spokes, 1 + (k + 1) * spokes
        e += [np.stack([a + i, b + i, b + j], 1), np.stack([a + i, b + j, a + j], 1)]
    fixed = np.zeros(1 + rings * spokes, dtype=bool)
    fixed[-spokes:] = True
    return np.concatenate(p), np.concatenate(e).astype(np.int32), fixed


def _mesh(name):
    if name == "wheel":
        return _wheel()
    if name.startswith("cube"):
        X, T, _ = W.kuhn_cube_mesh(int(name[4:]))
        return X, T, None
    X, T, _ = W.square_mesh(int(name[6:]), 0.3, cfg=3, item=1)
    return X, T, None


# unknowns: 64 (no smoothed auxiliary level), 1024, 1521, 8836; the cube's small levels
@pytest.mark.parametrize("name", ["square9", "square33", "square40", "square95", "wheel", "cube9"])
@pytest.mark.parametrize("sigma", [0.0, 0.5])
@pytest.mark.parametrize("nu", [(2, 1), (1, 2)])
def test_preconditioner(name, sigma, nu):
    X, T, fixed = _mesh(name)
    kappa = np.exp(sigma * np.random.default_rng(3).standard_normal(len(T)))
    H = Hierarchy(X, T, kappa, dirichlet=fixed, colouring="smallest_last")
    S = A.Solver(X, T, kappa, fixed, nu_aux=nu[0], nu_fine=nu[1])
    r = np.random.default_rng(4).standard_normal(H.n)
    z = H.preconditioner(nu_aux=nu[0], nu_fine=nu[1])(r)
    rd = torch.from_numpy(r).cuda()
    assert _rel_inf(S.apply_preconditioner(rd).cpu().numpy(), z) <= 1e-12
    assert _rel_inf(S.apply_preconditioner(rd, precision=A.PREC_MIXED).cpu().numpy(), z) <= 1e-5


@pytest.mark.parametrize("first", [0.0, 0.5])
def test_coefficient_update_changes_the_coding(first):
    X, T, _ = _mesh("square60")
    k = [np.exp(s * np.random.default_rng(3).standard_normal(len(T))) for s in (first, 0.5 - first, first)]
    S = A.Solver(X, T, k[0])
    f = torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, S.n)).cuda()
    S.solve_device(f, 1e-8)
    for kappa in k[1:]:
        S.update_coefficient(kappa)
        R = A.Solver(X, T, kappa)
        for precision in (A.PREC_FP64, A.PREC_MIXED):
            assert torch.equal(S.apply_preconditioner(f, precision), R.apply_preconditioner(f, precision))
        u, it, _ = S.solve_device(f, 1e-8)
        v, jt, _ = R.solve_device(f, 1e-8)
        assert it == jt and torch.equal(u, v)


# two and four right-hand sides (four FP64 values go as two blocks of two) on the same sizes in one batch; the
# bars of the batched parity tests: iterates within 1e-10 of the oracle's after the same number of steps
@pytest.mark.parametrize("nr", [2, 4])
@pytest.mark.parametrize("sigma", [0.0, 0.5])
def test_batched_right_hand_sides(nr, sigma):
    rng = np.random.default_rng(6)
    meshes, H, F = [], [], []
    for name in ("square9", "square33", "wheel", "square95"):
        X, T, _ = _mesh(name)
        kappa = np.exp(sigma * rng.standard_normal(len(T)))
        meshes.append((X, T, kappa))
        H.append(Hierarchy(X, T, kappa, colouring="smallest_last"))
        F.append(rng.standard_normal((nr, H[-1].n)))
    B = A.BatchSolver(meshes)
    U, its, _ = B.solve(torch.from_numpy(np.concatenate([f.ravel() for f in F])).cuda(), nr, 1e-8)
    U, off = U.cpu().numpy(), B.offsets(nr)
    for m, h in enumerate(H):
        u = U[off[m]:off[m + 1]].reshape(nr, h.n)
        for r in range(nr):
            v, it, info = h.solve(F[m][r], 1e-8, record=True)
            near = any(abs(x - 1e-8) < 1e-3 * 1e-8 for x in info["history"][-2:])
            assert its[m, r] == it or near
            if its[m, r] == it:
                assert np.linalg.norm(u[r] - v) <= 1e-10 * np.linalg.norm(v)


# the map from matrix entries to the patches' values, on the sizes above: the original grid's sweeps follow a
# coefficient set on the device, the auxiliary hierarchy keeps the first one
@pytest.mark.parametrize("name", ["square9", "square33", "square40", "square95", "wheel"])
def test_device_coefficient(name):
    X, T, fixed = _mesh(name)
    rng = np.random.default_rng(8)
    kappa = np.exp(0.5 * rng.standard_normal(len(T)))
    S = A.Solver(X, T, np.ones(len(T)), fixed)
    H = Hierarchy(X, T, np.ones(len(T)), dirichlet=fixed, colouring="smallest_last")
    H.A = Hierarchy(X, T, kappa, dirichlet=fixed, colouring="smallest_last").A
    r = rng.standard_normal(H.n)
    z = H.preconditioner(nu_aux=2, nu_fine=1)(r)
    S.set_coefficient_device(torch.from_numpy(kappa).cuda())
    rd = torch.from_numpy(r).cuda()
    assert _rel_inf(S.apply_preconditioner(rd).cpu().numpy(), z) <= 1e-12
    assert _rel_inf(S.apply_preconditioner(rd, precision=A.PREC_MIXED).cpu().numpy(), z) <= 1e-5
