"""Which levels run patches (csrc/patch.hpp), in which form, so that the parity tests of the patches cannot pass on
the colour passes alone; and B_co on 3-D meshes whose levels have patches, of the larger shape among them (FP64: 1e-12)."""
import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")

FIELDS = ("patches", "big", "matrix", "transfer", "fp64", "fp32")


def _patches(S, level):
    return dict(zip(FIELDS, S.export("patches", level).tolist()))


def _levels(S):
    i = S.info()
    return range(i["lc"] + 1, i["J"] + 1)


@pytest.mark.parametrize("n", [33, 95])
@pytest.mark.parametrize("sigma", [0.0, 0.5])
def test_square(n, sigma):
    X, T, _ = W.square_mesh(n, 0.3, cfg=3, item=1)
    S = A.Solver(X, T, np.exp(sigma * np.random.default_rng(3).standard_normal(len(T))))
    g = _patches(S, -1)
    assert g["patches"] >= 1 and g["fp64"] and g["fp32"] and not (g["big"] or g["matrix"] or g["transfer"])
    for l in _levels(S):
        p = _patches(S, l)
        assert p["patches"] >= 1 and p["fp64"] and p["fp32"] and p["transfer"] and not p["big"]
        assert p["matrix"] == (sigma == 0.0)
    with pytest.raises(A.AsmgError):
        S.export("patches", S.info()["J"] + 1)


def test_batch():
    meshes = []
    for n in (2, 9, 33, 95):
        X, T, _ = W.square_mesh(n, 0.3, cfg=3, item=n)
        meshes.append((X, T, np.ones(len(T))))
    B = A.BatchSolver(meshes)
    depth = int((B._export(b"batch_J", 0, np.int64) - B._export(b"batch_lc", 0, np.int64)).max())
    assert depth >= 1
    for k in range(-1, depth):
        p = dict(zip(FIELDS, B._export(b"batch_patches", k, np.int64).tolist()))
        assert p["patches"] >= 1 and p["fp64"] and p["fp32"] and not p["big"]
    assert B._export(b"batch_patches", depth, np.int64)[0] == 0  # bottom solves only


def _csr(S, name, shape, level=0):
    return sp.csr_matrix((S.export(name + "_val", level), S.export(name + "_col", level),
                          S.export(name + "_rowptr", level)), shape=shape)


def _sweeps(M, colour, x, b, nu, backward):
    rows = [np.flatnonzero(colour == c) for c in range(int(colour.max()) + 1)]
    parts = [(r, M[r], M.diagonal()[r]) for r in (rows[::-1] if backward else rows)]
    for _ in range(nu):
        for r, Mr, d in parts:
            x[r] += (b[r] - Mr @ x) / d
    return x


def _preconditioner(S, b, nu_aux, nu_fine):
    """Algorithms 1 and 2 on the exported matrices, transfers, colours and bottom inverse, in scipy."""
    i = S.info()
    n = {l: len(S.export("Al_rowptr", l)) - 1 for l in range(i["lc"], i["J"] + 1)}

    def cycle(M, colour, T, nu, b, below):
        x = _sweeps(M, colour, np.zeros(len(b)), b, nu, False)
        x += T @ below(T.T @ (b - M @ x))
        return _sweeps(M, colour, x, b, nu, True)

    def level(l, b):
        if l == i["lc"]:
            return S.export("coarse_inv").reshape(n[l], n[l]) @ b
        return cycle(_csr(S, "Al", (n[l], n[l]), l), S.export("colour_aux", l), _csr(S, "P", (n[l], n[l - 1]), l), nu_aux,
                     b, lambda g: level(l - 1, g))

    return cycle(_csr(S, "A", (S.n, S.n)), S.export("colour_fine"), _csr(S, "Pi", (S.n, n[i["J"]])), nu_fine, b,
                 lambda g: level(i["J"], g))


# patches of both shapes on 3-D levels of two to seven colours (the larger one from 31^3 cells on)
@pytest.mark.parametrize("n", [20, 31])
def test_cube(n):
    X, T, _ = W.kuhn_cube_mesh(n, item=1)
    S = A.Solver(X, T, np.exp(0.5 * np.random.default_rng(n).standard_normal(len(T))))
    levels = [_patches(S, l) for l in _levels(S)]
    assert all(p["patches"] >= 2 and p["fp64"] and not p["fp32"] for p in levels)
    assert any(p["big"] for p in levels) == (n == 31)
    r = np.random.default_rng(4).standard_normal(S.n)
    z = _preconditioner(S, r, 2, 1)
    got = S.apply_preconditioner(torch.from_numpy(r).cuda()).cpu().numpy()
    assert np.abs(got - z).max() <= 1e-12 * np.abs(z).max()
