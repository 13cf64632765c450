"""Handles of other sizes on other threads run the same patch kernels (four FP64 right-hand sides, 3-D levels: more
than 64 KiB of LDS): the results are those of one thread."""
import threading

import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


def _handle(sides):
    if len(sides) == 1:
        X, T, _ = W.kuhn_cube_mesh(sides[0])
        S = A.Solver(X, T, np.ones(len(T)))
        return lambda f: S.solve_device(f, 1e-8)[0], S.n
    B = A.BatchSolver([(X, T, np.ones(len(T))) for X, T, _ in (W.square_mesh(n, 0.3, cfg=3, item=n) for n in sides)])
    return lambda f: B.solve(f, 4, 1e-8)[0], 4 * B.n_total


def test_threads():
    work = [(12, 16), (90, 120, 70), (40,), (24,)]
    want, first, f = [], [], []
    for w in work:
        solve, n = _handle(w)
        f.append(torch.from_numpy(np.random.default_rng(1).uniform(-1, 1, n)).cuda())
        want.append(solve(f[-1]))
        first.append(_handle(w)[0])  # its first solves run on a thread
    torch.cuda.synchronize()
    got = [None] * len(work)

    def run(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            got[i] = [first[i](f[i]) for _ in range(3)]

    threads = [threading.Thread(target=run, args=(i,)) for i in range(len(work))]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for w, g, u in zip(work, got, want):
        assert g is not None and all(torch.equal(v, u) for v in g), w
