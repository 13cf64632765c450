"""Host coefficient updates of patched levels: new values go to the stored places of the old ones, so the handle has to
give the same bits as one that was set up with them. Rows longer than the entries kept in registers, both patch
shapes, matrices that stay coded with other values, and an update after a coefficient that was set on the device."""
import numpy as np
import pytest

import workloads as W
from test_gpu_patch import _wheel

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


def _mesh(name):
    if name == "wheel":
        return _wheel()
    n = int(name.split()[1])
    return (*(W.kuhn_cube_mesh(n) if name.startswith("cube") else W.square_mesh(n, 0.3, cfg=3, item=1))[:2], None)


@pytest.mark.parametrize("name", ["wheel", "square 41", "square 150", "cube 17", "cube 36"])
def test_update_equals_setup(name):
    X, T, fixed = _mesh(name)
    rng = np.random.default_rng(3)
    one, rough, other = np.ones(len(T)), np.exp(0.5 * rng.standard_normal(len(T))), np.exp(rng.standard_normal(len(T)))
    S = A.Solver(X, T, one, fixed)
    f = torch.from_numpy(rng.uniform(-1, 1, S.n)).cuda()
    for i, kappa in enumerate((rough, other, 3.0 * one, one, rough)):
        if i == 1:
            S.set_coefficient_device(torch.from_numpy(one).cuda())
        S.update_coefficient(kappa)
        R = A.Solver(X, T, kappa, fixed)
        for precision in (A.PREC_FP64, A.PREC_MIXED):
            assert torch.equal(S.apply_preconditioner(f, precision), R.apply_preconditioner(f, precision)), (i, precision)
        u, it, _ = S.solve_device(f, 1e-8)
        v, jt, _ = R.solve_device(f, 1e-8)
        assert it == jt and torch.equal(u, v)
