"""The patch layout (csrc/patch.hpp) on the CPU: tests/patch_check_main.hip lays a level out and runs the patch
kernels' steps on an LDS image that starts as NaN, so a cell that is read before it is written, or a row that
reads another mesh's cell, shows in the result. Compared with plain sweeps over the whole level.

Bar: 1e-12 of the largest value (a few dozen FP64 operations a row, sums in another order)."""
import os
import shutil
import subprocess

import numpy as np
import pytest
import scipy.sparse as sp

import workloads as W

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
CSRC = os.path.join(ROOT, "paper_1410_2153_amd", "csrc")
HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

pytestmark = pytest.mark.skipif(shutil.which(HIPCC) is None, reason="needs hipcc")


@pytest.fixture(scope="module")
def exe(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("patch") / "patch_check")
    src = os.path.join(os.path.dirname(os.path.abspath(__file__)), "patch_check_main.hip")
    subprocess.run([HIPCC, "-x", "hip", "--offload-arch=gfx950", "-std=c++17", "-O1", "-w", "-Xclang", "-target-feature",
                    "-Xclang", "-packed-fp32-ops", "-I" + CSRC, "-I" + os.path.join(ROOT, "include"), src, "-o", out,
                    "-lpthread"], check=True)
    return out


def _level(meshes, seed):
    """Block matrix of (coords, elems, Dirichlet mask) meshes: A without its diagonal, the diagonal, colours, spatial
    order, the mesh of each row, and a prolongation of up to three entries a row (some rows have none) inside each
    mesh."""
    r = np.random.default_rng(seed)
    A, diag, order, mesh, P, off, coff = [], [], [], [], [], 0, 0
    for m, (X, T, fixed) in enumerate(meshes):
        free = np.flatnonzero(~fixed)
        num = np.full(len(X), -1)
        num[free] = np.arange(len(free))
        i = np.concatenate([T[:, a] for a in range(3) for b in range(3) if a != b])
        j = np.concatenate([T[:, b] for a in range(3) for b in range(3) if a != b])
        keep = (num[i] >= 0) & (num[j] >= 0)
        B = sp.csr_matrix((np.ones(keep.sum()), (num[i[keep]], num[j[keep]])), shape=(len(free),) * 2)
        B = sp.triu(B, 1).tocsr()
        B.data = -r.uniform(0.5, 1.0, len(B.data))
        B = (B + B.T).tocsr()
        B.sort_indices()
        A.append(B)
        diag.append(1.0 + np.asarray(np.abs(B).sum(1)).ravel())
        q = (X[free] * 1023).astype(int)
        key = sum(((q[:, d] >> b & 1) << (2 * b + d)) for d in range(2) for b in range(10))
        order.append(off + np.argsort(key, kind="stable"))
        mesh.append(np.full(len(free), m))
        nc = max(1, len(free) // 4)
        i = np.repeat(np.arange(len(free)), 3)
        j = np.argsort(order[-1]).repeat(3) // 4 + np.tile([-1, 0, 1], len(free))
        keep = (r.random(len(i)) < 0.5) & (j >= 0) & (j < nc)
        P.append(sp.csr_matrix((r.choice([1.0, 0.5], keep.sum()), (i[keep], j[keep])), shape=(len(free), nc)))
        off += len(free)
        coff += nc
    A = sp.block_diag(A).tocsr()
    P = sp.block_diag(P).tocsr()
    for M in (A, P):
        M.sort_indices()
    col = np.full(off, -1)
    for i in range(off):
        used = set(col[A.indices[A.indptr[i]:A.indptr[i + 1]]])
        col[i] = next(c for c in range(64) if c not in used)
    return A, np.concatenate(diag), col, np.concatenate(order), np.concatenate(mesh), P


def _reference(A, diag, col, P, b, e, nu):
    C = col.max() + 1
    x = np.zeros(len(b))
    rows = [np.flatnonzero(col == c) for c in range(C)]
    with np.errstate(all="ignore"):
        for s in range(nu):
            for c in range(C):
                x[rows[c]] = (b[rows[c]] - A[rows[c]] @ x) / diag[rows[c]]
        r = b - diag * x - A @ x
        r[rows[-1]] = 0.0
        y = x + P @ e
        for s in range(nu):
            for c in range(C - 1, -1, -1):
                y[rows[c]] = (b[rows[c]] - A[rows[c]] @ y) / diag[rows[c]]
    return x, P.T @ r, y


def _run(exe, tmp_path, level, b, e, nu, own, shape):
    A, diag, col, order, _, P = level
    n, nc = A.shape[0], P.shape[1]
    path, out = str(tmp_path / "in.bin"), str(tmp_path / "out.bin")
    with open(path, "wb") as f:
        np.array([n, col.max() + 1, nu, nc, own, shape], np.int32).tofile(f)
        for M in (A,):
            M.indptr.astype(np.int32).tofile(f), M.indices.astype(np.int32).tofile(f), M.data.tofile(f)
        diag.tofile(f), col.astype(np.int32).tofile(f), order.astype(np.int32).tofile(f)
        P.indptr.astype(np.int32).tofile(f), P.indices.astype(np.int32).tofile(f), P.data.tofile(f)
        b.tofile(f), e.tofile(f)
    subprocess.run([exe, path, out], check=True, timeout=300)
    v = np.fromfile(out, np.float64, 2 * n + nc)
    npatch, alone = np.fromfile(out, np.int32, offset=8 * (2 * n + nc))
    return v[:n], v[n:n + nc], v[n + nc:], int(npatch), int(alone)


def _isolate(X, T, fixed, count, seed):
    """Dirichlet values on every neighbour of `count` scattered vertices: unknowns without neighbours."""
    r = np.random.default_rng(seed)
    fixed = fixed.copy()
    nb = sp.csr_matrix((np.ones(9 * len(T)), (T.repeat(3, 1).ravel(), np.tile(T, (1, 3)).ravel())), shape=(len(X),) * 2)
    for v in r.choice(np.flatnonzero(~fixed), count, replace=False):
        if fixed[v]:
            continue
        near = nb.indices[nb.indptr[v]:nb.indptr[v + 1]]
        fixed[near[near != v]] = True
        fixed[v] = False
    return fixed


def _square(n, isolated=0, seed=0):
    X, T, _ = W.square_mesh(n, 0.3, cfg=3, item=seed)
    T = np.asarray(T)
    fixed = (X == 0).any(1) | (X == 1).any(1)
    return X, T, _isolate(X, T, fixed, isolated, seed) if isolated else fixed


# unknowns without neighbours inside a mesh of several patches, both shapes, one and two sweeps
@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("shape", [0, 1])
@pytest.mark.parametrize("seed", [0, 1, 2])
def test_rows_without_neighbours(exe, tmp_path, nu, shape, seed):
    level = _level([_square(120, 150, seed)], seed)
    A, diag, col, _, _, P = level
    assert (np.diff(A.indptr) == 0).sum() >= 100
    r = np.random.default_rng(10 + seed)
    b, e = r.standard_normal(A.shape[0]), r.standard_normal(P.shape[1])
    x, bc, xo, npatch, alone = _run(exe, tmp_path, level, b, e, nu, 400, shape)
    assert npatch > 5
    for got, want in zip((x, bc, xo), _reference(A, diag, col, P, b, e, nu)):
        assert np.abs(got - want).max() <= 1e-12 * np.abs(want).max()


# a NaN in one mesh of a batch stays there: one-unknown meshes share patches with it
@pytest.mark.parametrize("nu", [1, 2])
@pytest.mark.parametrize("bad", [0, 2])
def test_meshes_stay_apart(exe, tmp_path, nu, bad):
    level = _level([_square(20, 0, 0), _square(2), _square(12, 4, 1), _square(2), _square(3)], 5)
    A, diag, col, _, mesh, P = level
    r = np.random.default_rng(11)
    b, e = r.standard_normal(A.shape[0]), r.standard_normal(P.shape[1])
    want = _reference(A, diag, col, P, b, e, nu)
    b[mesh == bad] = np.nan
    cmesh = np.asarray(mesh[sp.csc_matrix(P).indices[np.minimum(sp.csc_matrix(P).indptr[:-1], P.nnz - 1)]])
    cmesh[np.diff(sp.csc_matrix(P).indptr) == 0] = -1
    e[cmesh == bad] = np.nan
    got = _run(exe, tmp_path, level, b, e, nu, A.shape[0], 0)
    assert got[3] == 1
    for v, w, m in zip(got, want, (mesh, cmesh, mesh)):
        assert np.abs(v - w)[m != bad].max() <= 1e-12 * np.abs(w).max()
