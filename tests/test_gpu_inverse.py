"""The bottom inverse built on the device (csrc/inverse.hpp) against the host's, at sizes around its blocks of 32
and tiles of 64 unknowns, a regularised one (pure Neumann) included.

Bar: |A X - I| element-wise within 64 eps cond-free growth, n eps max|A| max|X| with eps = 2^-52 (a backward stable
elimination of an SPD matrix), and the host's inverse to the same bound relative to max|X|^2 max|A|.
"""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


# coarse_max_dofs picks the bottom: 1, 9, 49, 225, 961 unknowns on squares; the annulus is pure Neumann
@pytest.mark.parametrize("case", [("square", 1), ("square", 9), ("square", 49), ("square", 225), ("square", 961),
                                  ("annulus", 1024)])
def test_inverse(case):
    kind, most = case
    kw = dict(coarse_max_dofs=most)
    if kind == "square":
        X, T, _ = W.square_mesh(40, 0.3, cfg=3, item=1)
    else:
        X, T, _ = W.annulus_mesh(160)
        kw.update(domain=2, dirichlet=np.zeros(len(X), dtype=bool))
    kappa = np.exp(0.5 * np.random.default_rng(3).standard_normal(len(T)))
    D = A.Solver(X, T, kappa, **kw)
    H = A.Solver(X, T, kappa, device=-1, **kw)
    lc = D.info()["lc"]
    n = int(D.export("level_n")[lc - 1])
    d = D.export("coarse_inv").reshape(n, n)
    h = H.export("coarse_inv").reshape(n, n)
    M = H.export_csr("Al", lc, shape=(n, n)).toarray()
    eps = 2.0 ** -52
    if kind == "square":
        assert np.abs(M @ d - np.eye(n)).max() <= 8 * n * eps * np.abs(M).max() * np.abs(d).max()
    assert np.abs(d - h).max() <= 8 * n * eps * np.abs(M).max() * np.abs(d).max() ** 2
    # a new coefficient replaces it
    k2 = kappa[::-1].copy()
    D.update_coefficient(k2)
    h2 = A.Solver(X, T, k2, device=-1, **kw).export("coarse_inv").reshape(n, n)
    assert np.abs(D.export("coarse_inv").reshape(n, n) - h2).max() <= 8 * n * eps * np.abs(M).max() * np.abs(h2).max() ** 2 * 4
