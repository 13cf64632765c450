"""Device memory of a handle whose coefficient changes between constant (matrix values as codes) and variable: what a
level has held in either form is used again."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


def test_changing_the_coding_does_not_grow():
    X, T, _ = W.square_mesh(400, 0.3, cfg=3, item=1)
    k = [np.ones(len(T)), np.exp(0.5 * np.random.default_rng(3).standard_normal(len(T)))]
    S = A.Solver(X, T, k[0], setup_device=1)
    f = torch.from_numpy(np.random.default_rng(5).uniform(-1, 1, S.n)).cuda()
    free = []
    for i in range(8):
        S.update_coefficient(k[(i + 1) % 2])
        S.solve_device(f, 1e-8)
        torch.cuda.synchronize()
        free.append(torch.cuda.mem_get_info()[0])
    # one round of both forms may allocate; its graphs are captured again at each change
    assert free[1] - min(free[2:]) <= 4 << 20, free
