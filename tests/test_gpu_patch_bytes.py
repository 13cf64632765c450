"""The byte model of the patch launches: coded entries move their cell or column number only, so on one mesh a
constant coefficient (coded level matrices) and a varying one (plain values) differ by the values of those levels'
off-diagonal entries, once in each of a level's two launches."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


@pytest.mark.parametrize("precision, size", [(A.PREC_FP64, 8), (A.PREC_MIXED, 4)])
def test_coded_values_are_not_counted(precision, size):
    X, T, _ = W.square_mesh(95, 0.3, cfg=3, item=1)
    kappa = np.exp(0.5 * np.random.default_rng(3).standard_normal(len(T)))
    coded, plain = A.Solver(X, T, np.ones(len(T))), A.Solver(X, T, kappa)
    i = coded.info()
    entries = 0
    for l in range(i["lc"] + 1, i["J"] + 1):
        a, b = coded.export("patches", l), plain.export("patches", l)
        assert a[0] == b[0] > 0 and a[2] == 1 and b[2] == 0
        rp = coded.export("Al_rowptr", l)
        entries += int(rp[-1]) - (len(rp) - 1)
    assert entries > 0
    by = [S.time_kernel(2, reps=1, precision=precision)[1] for S in (coded, plain)]
    assert by[1] - by[0] == 2 * entries * size


@pytest.mark.parametrize("precision, size", [(A.PREC_FP64, 8), (A.PREC_MIXED, 4)])
def test_batch(precision, size):
    X, T, _ = W.square_mesh(95, 0.3, cfg=3, item=1)
    kappa = np.exp(0.5 * np.random.default_rng(3).standard_normal(len(T)))
    one = A.Solver(X, T, np.ones(len(T)), device=-1)
    i = one.info()
    entries = 0
    for l in range(i["lc"] + 1, i["J"] + 1):
        rp = one.export("Al_rowptr", l)
        entries += int(rp[-1]) - (len(rp) - 1)
    by = [A.BatchSolver([(X, T, k)]).time_kernel(0, 4, reps=1, precision=precision)[1]
          for k in (np.ones(len(T)), kappa)]
    assert by[1] - by[0] == 2 * entries * size
