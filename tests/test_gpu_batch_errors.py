"""A batch whose bottom matrix is not positive definite is refused with the mesh that has it."""
import numpy as np
import pytest

import workloads as W

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")
A = pytest.importorskip("paper_1410_2153_amd")


@pytest.mark.parametrize("bad", [0, 1, 2])
def test_the_error_names_the_mesh(bad):
    meshes = []
    for i, n in enumerate((40, 12, 70)):
        X, T, _ = W.square_mesh(n, 0.3, cfg=3, item=i)
        meshes.append((X, T, np.full(len(T), 1e308 if i == bad else 1.0)))  # the entries overflow
    for device in (-1, 0):
        with pytest.raises(A.AsmgError, match=f"mesh {bad}: matrix of an exact subsystem solve"):
            A.BatchSolver(meshes, device=device)
