"""Unknowns without neighbours (every neighbour on the Dirichlet boundary, or the single unknown of a 2 x 2 square in
a batch): their rows share patches with longer rows and with other meshes.

Bars as in the other parity tests: B_co element-wise within 1e-12 (FP64) and 1e-5 (FP32 V-cycle) of the oracle's;
the systems of a batch do not depend on each other, so they are the same bits whatever another mesh's values are."""
import numpy as np
import pytest

import workloads as W
from oracle.hierarchy import Hierarchy
from test_patch_layout import _square

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


@pytest.mark.parametrize("nu_fine", [1, 2])
def test_isolated_unknowns(nu_fine):
    X, T, fixed = _square(120, 150, 2)
    kappa = np.exp(0.5 * np.random.default_rng(3).standard_normal(len(T)))
    H = Hierarchy(X, T, kappa, dirichlet=fixed, colouring="smallest_last")
    assert ((H.A != 0).sum(1) == 1).sum() >= 100
    S = A.Solver(X, T, kappa, fixed, nu_fine=nu_fine)
    r = np.random.default_rng(4).standard_normal(H.n)
    z = H.preconditioner(nu_aux=2, nu_fine=nu_fine)(r)
    rd = torch.from_numpy(r).cuda()
    # leaves NaN in the LDS of the CUs
    with pytest.raises(A.AsmgError):
        S.solve_device(torch.full_like(rd, float("nan")), 1e-8)
    for precision, bar in ((A.PREC_FP64, 1e-12), (A.PREC_MIXED, 1e-5)):
        got = S.apply_preconditioner(rd, precision=precision).cpu().numpy()
        assert np.abs(got - z).max() <= bar * np.abs(z).max()


@pytest.mark.parametrize("nr", [1, 4])
@pytest.mark.parametrize("bad", [0, 2])
def test_nan_stays_in_its_mesh(nr, bad):
    rng = np.random.default_rng(6)
    meshes = []
    for i, n in enumerate((20, 2, 33, 2, 3)):
        X, T, _ = W.square_mesh(n, 0.3, cfg=3, item=i)
        meshes.append((X, T, np.exp(0.5 * rng.standard_normal(len(T)))))
    B = A.BatchSolver(meshes)
    off = B.offsets(nr)
    f = torch.from_numpy(rng.standard_normal(off[-1])).cuda()
    want, _, _ = B.solve(f, nr, 1e-8)
    assert want.isfinite().all()
    f[off[bad]:off[bad + 1]] = float("nan")
    got = torch.full_like(f, 7.0)
    with pytest.raises(A.AsmgError):
        B.solve(f, nr, 1e-8, out=got)
    for m in range(len(meshes)):
        if m != bad:
            assert torch.equal(got[off[m]:off[m + 1]], want[off[m]:off[m + 1]]), m
