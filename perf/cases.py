"""The solver's work as a user's program asks for it: a list of timed cases, and draws of the same ranges.

A case is a dict of plain values. Its meshes, coefficients and right-hand sides come from the seed:

* ``square``  -- n x n cells of the unit square, random diagonals, jittered interior nodes, Dirichlet boundary
* ``graded``  -- the same grid pulled radially towards the corner (0, 0), mesh size growing like sqrt(r)
* ``annulus`` -- 1/5 <= r <= 1/2, a Dirichlet outer circle and a Neumann hole (general-domain grids)
* ``cube``    -- n^3 cells of six Kuhn tetrahedra, jittered, coefficient {1, 10} on a checkerboard

Kinds of call: ``solve`` (one mesh, one right-hand side), ``oneshot`` (a new mesh: setup, then one solve of
a host vector), ``batch`` (many meshes with up to 4 right-hand sides each), ``krylov`` (the preconditioner
and the matrix product, as a program with its own Krylov loop calls them) and ``gradient`` (the gradient of
a misfit with respect to the log-coefficients, through autograd).
"""
from __future__ import annotations

import math

import numpy as np
import torch

import paper_1410_2153_amd as A

TOL = 1e-8


def listed():
    return [
        # the smallest useful problem, solved from device memory: launches and latency only
        dict(name="solve square 32", kind="solve", mesh="square", n=32, precision="fp64", sigma=0.0, host=False),
        # the small workload of the benchmark (64 x 64, coefficient 1), vectors on the host
        dict(name="solve square 64 host", kind="solve", mesh="square", n=64, precision="fp64", sigma=0.0, host=True),
        # a locally refined mesh of ordinary size with a rough coefficient
        dict(name="solve graded 350", kind="solve", mesh="graded", n=350, precision="fp64", sigma=0.5, host=False),
        # the same at the benchmark's million unknowns, with the FP32 preconditioner
        dict(name="solve graded 1001 mixed", kind="solve", mesh="graded", n=1001, precision="mixed", sigma=0.5, host=False),
        # tetrahedra, both precisions; the second with an odd number of cells
        dict(name="solve cube 64", kind="solve", mesh="cube", n=64, precision="fp64", sigma=0.0, host=False),
        dict(name="solve cube 31 mixed", kind="solve", mesh="cube", n=31, precision="mixed", sigma=0.0, host=False),
        # many meshes at once: small ones with one right-hand side, the benchmark's sides with four and two
        dict(name="batch small x1", kind="batch", meshes=48, lo=8, hi=64, rhs=1, precision="fp64"),
        dict(name="batch wide x4", kind="batch", meshes=40, lo=32, hi=512, rhs=4, precision="fp64"),
        dict(name="batch wide x2 mixed", kind="batch", meshes=25, lo=32, hi=511, rhs=2, precision="mixed"),
        # a program with its own Krylov loop on a domain with a hole
        dict(name="krylov annulus 200", kind="krylov", mesh="annulus", n=200, precision="fp64", sigma=0.5),
        # the adjoint workload: refresh of A, forward solve, adjoint solve, element gradients
        dict(name="gradient square 500", kind="gradient", mesh="square", n=500, precision="fp64", sigma=0.3),
        # a mesh that is solved once: the setup and the first solve are all there is
        dict(name="oneshot square 100", kind="oneshot", mesh="square", n=100, precision="fp64", sigma=0.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "solve", "batch", "batch", "krylov", "gradient", "oneshot"])
    precision = rng.choice(["fp64", "fp64", "mixed"])
    if kind == "batch":
        lo = _log_int(rng, 8, 64)
        hi = _log_int(rng, lo + 8, 512)
        most = 1_000_000 / (((lo + hi) / 2) ** 2 + (hi - lo) ** 2 / 12)  # unknowns of the batch
        return dict(kind=kind, meshes=max(2, min(64, int(most * rng.uniform(0.3, 1.0)))), lo=lo, hi=hi,
                    rhs=rng.choice([1, 2, 4]), precision=precision)
    mesh = rng.choice(["square", "graded", "annulus", "cube"] if kind in ("solve", "krylov") else ["square", "graded"])
    n = {"square": (16, 1000), "graded": (24, 1000), "annulus": (24, 300), "cube": (8, 64)}[mesh]
    n = _log_int(rng, n[0], {"gradient": 500, "oneshot": 250}.get(kind, n[1]))
    sigma = 0.0 if mesh == "cube" else rng.choice([0.0, 0.3, 0.5])
    if kind == "gradient":
        sigma = max(sigma, 0.3)
    case = dict(kind=kind, mesh=mesh, n=n, precision=precision, sigma=sigma)
    if kind == "solve":
        case["host"] = rng.random() < 0.25
    return case


# ------------------------------------------------------------------------------------------------------
# meshes
# ------------------------------------------------------------------------------------------------------


def _grid2(nx, ny, r):
    """Triangles of an nx x ny grid of cells, each cut along a random diagonal; vertex (i, j) is i + j (nx + 1)."""
    v = np.arange((nx + 1) * (ny + 1), dtype=np.int32).reshape(ny + 1, nx + 1)
    a, b, c, d = (q.ravel() for q in (v[:-1, :-1], v[:-1, 1:], v[1:, :-1], v[1:, 1:]))
    flip = (r.random(nx * ny) < 0.5)[:, None]
    t = np.empty((2 * nx * ny, 3), dtype=np.int32)
    t[0::2] = np.where(flip, np.stack([a, b, c], 1), np.stack([a, b, d], 1))
    t[1::2] = np.where(flip, np.stack([b, d, c], 1), np.stack([a, d, c], 1))
    return t


def _cells2(nx, ny, r, jitter):
    """Grid points in units of cells, interior ones jittered, and a mask of the boundary."""
    y, x = np.meshgrid(np.arange(ny + 1.0), np.arange(nx + 1.0), indexing="ij")
    p = np.stack([x.ravel(), y.ravel()], 1)
    edge = (p[:, 0] == 0) | (p[:, 0] == nx) | (p[:, 1] == 0) | (p[:, 1] == ny)
    p[~edge] += r.uniform(-jitter, jitter, (int((~edge).sum()), 2))
    return p, edge


def _mesh(kind, n, seed):
    """(coords, elems, Dirichlet mask, coefficient pattern or None, the general domain option)."""
    r = np.random.default_rng([int(seed), 1, int(n)])
    if kind in ("square", "graded"):
        p, edge = _cells2(n, n, r, 0.2)
        p /= n
        if kind == "graded":
            p *= np.sqrt(p.max(axis=1))[:, None]
        return p, _grid2(n, n, r), edge, None, 0
    if kind == "annulus":  # n rings of 5 n cells
        nx = 5 * n
        p, _ = _cells2(nx, n, r, 0.15)
        t = 2 * np.pi * p[:, 0] / nx
        s = 0.2 + 0.3 * p[:, 1] / n
        p = np.stack([0.5 + s * np.cos(t), 0.5 + s * np.sin(t)], 1)
        e = _grid2(nx, n, r)
        v = np.arange((nx + 1) * (n + 1))
        i, j = v % (nx + 1), v // (nx + 1)
        p = p[i < nx]
        e = ((i % nx) + j * nx)[e].astype(np.int32)
        outer = np.zeros(len(p), dtype=bool)
        outer[n * nx:] = True
        return p, e, outer, None, 2
    g = np.arange(n + 1.0)
    z, y, x = np.meshgrid(g, g, g, indexing="ij")
    p = np.stack([x.ravel(), y.ravel(), z.ravel()], 1)
    edge = ((p == 0) | (p == n)).any(1)
    p[~edge] += r.uniform(-0.15, 0.15, (int((~edge).sum()), 3))
    k, j, i = (q.ravel() for q in np.meshgrid(np.arange(n), np.arange(n), np.arange(n), indexing="ij"))
    step = [1, n + 1, (n + 1) ** 2]
    base = i + (n + 1) * (j + (n + 1) * k)
    e = np.empty((6 * n ** 3, 4), dtype=np.int32)
    for q, (a, b, _) in enumerate(((0, 1, 2), (0, 2, 1), (1, 0, 2), (1, 2, 0), (2, 0, 1), (2, 1, 0))):
        e[q::6] = np.stack([base, base + step[a], base + step[a] + step[b], base + sum(step)], 1)
    w = max(1, n // 8)
    kappa = np.where((i // w + j // w + k // w) % 2 == 0, 10.0, 1.0).repeat(6)
    return p / n, e, edge, kappa, 0


def _problem(case, seed):
    """Host arrays of a one-mesh case: coords, elems, Dirichlet mask, log-coefficient, right-hand side, domain."""
    p, e, fixed, kappa, domain = _mesh(case["mesh"], case["n"], seed)
    r = np.random.default_rng([int(seed), 2, int(case["n"])])
    m = np.log(kappa) if kappa is not None else case["sigma"] * r.standard_normal(len(e))
    f = r.uniform(-1.0, 1.0, int((~fixed).sum()))
    return p, e, fixed, m, f, domain


def _sides(case, seed):
    """Spread evenly over the range on a logarithmic scale, odd ones among them, whatever the seed."""
    k = case["meshes"]
    return [int(round(case["lo"] * (case["hi"] / case["lo"]) ** (i / max(1, k - 1)))) for i in range(k)]


def _precision(case):
    return A.PREC_MIXED if case["precision"] == "mixed" else A.PREC_FP64


def _unknowns(case):
    n = case["n"]
    return {"square": (n - 1) ** 2, "graded": (n - 1) ** 2, "annulus": 5 * n * n, "cube": (n - 1) ** 3}[case["mesh"]]


def _batch_meshes(case, seed):
    for i, n in enumerate(_sides(case, seed)):
        p, e, fixed, _, _ = _mesh("square", n, seed * 1000 + i)
        yield p, e, fixed


# ------------------------------------------------------------------------------------------------------
# a program's state, and one pass
# ------------------------------------------------------------------------------------------------------


def prepare(case, seed):
    kind = case["kind"]
    if kind == "batch":
        meshes = [(p, e, np.ones(len(e))) for p, e, _ in _batch_meshes(case, seed)]
        solver = A.BatchSolver(meshes, precision=_precision(case))
        r = np.random.default_rng([int(seed), 2, case["meshes"]])
        f = r.uniform(-1.0, 1.0, solver.n_total * case["rhs"])
        return dict(kind=kind, solver=solver, f=torch.from_numpy(f).cuda(), rhs=case["rhs"])
    p, e, fixed, m, f, domain = _problem(case, seed)
    options = dict(precision=_precision(case), domain=domain)
    if domain:
        options["dirichlet"] = fixed
    if kind == "oneshot":
        return dict(kind=kind, mesh=(p, e, np.exp(m)), options=options, f=f)
    # programs that keep a mesh of some size build it on the device
    options["setup_device"] = 1
    if kind == "gradient":
        solver = A.Solver(p, e, np.ones(len(e)), **options)
        r = np.random.default_rng([int(seed), 3, case["n"]])
        seen = 1e-3 * r.standard_normal(solver.n)
        return dict(kind=kind, solver=solver, f=torch.from_numpy(f).cuda(), m=torch.from_numpy(m).cuda(),
                    seen=torch.from_numpy(seen).cuda(), function=A.LogCoefficientSolve.function())
    solver = A.Solver(p, e, np.exp(m), **options)
    host = kind == "solve" and case["host"]
    return dict(kind=kind, solver=solver, host=host, f=f if host else torch.from_numpy(f).cuda())


def run(state):
    kind = state["kind"]
    if kind == "batch":
        u, iterations, _ = state["solver"].solve(state["f"], state["rhs"], TOL)
        return [u, iterations]
    if kind == "oneshot":
        coords, elems, kappa = state["mesh"]
        solver = A.Solver(coords, elems, kappa, **state["options"])
        u, iterations, _ = solver.solve(state["f"], TOL)
        solver.close()
        return [u, iterations]
    solver = state["solver"]
    if kind == "krylov":
        z = solver.apply_preconditioner(state["f"])
        return [z, solver.matvec(z)]
    if kind == "gradient":
        m = state["m"].detach().requires_grad_(True)
        u = state["function"].apply(m, state["f"], solver, TOL)
        loss = 0.5 * (u - state["seen"]).square().sum()
        loss.backward()
        return [u.detach(), m.grad]
    # the third result, the true residual, is what is left of f - A u after the stopping rule: some digits
    # of it are rounding, so it is a check for the caller and no value to compare
    solve = solver.solve if state["host"] else solver.solve_device
    u, iterations, _ = solve(state["f"], TOL)
    return [u, iterations]


# ------------------------------------------------------------------------------------------------------
# what a pass cannot do without
# ------------------------------------------------------------------------------------------------------

STEPS = 8       # PCG steps that a residual of 1e-8 takes at least
ROW2, ROW3 = 6, 12  # entries of a row beside its diagonal


def work(case):
    """A PCG step reads the matrix once for the product and its preconditioner cannot do with less than one
    more pass over it; each reads and writes a handful of vectors."""
    kind = case["kind"]
    if kind == "batch":
        n = sum((s - 1) ** 2 for s in _sides(case, 0))
        rhs, row, steps = case["rhs"], ROW2, STEPS
    else:
        n, rhs, row = _unknowns(case), 1, ROW3 if case["mesh"] == "cube" else ROW2
        steps = {"krylov": 1, "gradient": 2 * STEPS}.get(kind, STEPS)
    value = 4 if case["precision"] == "mixed" else 8
    matrix = n * ((row + 1) * (8 + 4) + (row + 1) * (value + 4))
    vectors = n * rhs * (8 * 8 + 4 * value)
    return {"bytes": float(steps * (matrix + vectors)), "flops": float(steps * n * rhs * (4 * (row + 1) + 20))}


# ------------------------------------------------------------------------------------------------------
# the same in plain 64-bit arithmetic
# ------------------------------------------------------------------------------------------------------


class _Plain:
    """P1 stiffness matrix of a mesh in plain torch, and a Jacobi-preconditioned CG with it."""

    def __init__(self, p, e, fixed, kappa):
        p, e = torch.from_numpy(p).cuda(), torch.from_numpy(np.asarray(e, dtype=np.int64)).cuda()
        d = p.shape[1]
        self.kappa = torch.from_numpy(kappa).cuda()
        edges = p[e[:, 1:]] - p[e[:, :1]]
        inverse = torch.linalg.inv(edges)                       # columns: gradients of the last d hats
        g = torch.cat([-inverse.sum(2, keepdim=True), inverse], 2)
        size = torch.linalg.det(edges).abs() / math.factorial(d)
        self.k1 = sum(g[:, c, :, None] * g[:, c, None, :] for c in range(d)) * size[:, None, None]
        number = torch.full((len(p),), -1, dtype=torch.int64, device="cuda")
        free = torch.from_numpy(~fixed).cuda()
        self.n = int(free.sum())
        number[free] = torch.arange(self.n, device="cuda")
        self.dof = number[e]
        i = self.dof.unsqueeze(2).expand(-1, -1, d + 1).reshape(-1)
        j = self.dof.unsqueeze(1).expand(-1, d + 1, -1).reshape(-1)
        v = (self.k1 * self.kappa[:, None, None]).reshape(-1)
        keep = (i >= 0) & (j >= 0)
        a = torch.sparse_coo_tensor(torch.stack([i[keep], j[keep]]), v[keep], (self.n, self.n)).coalesce()
        at = a.indices()
        self.diagonal = torch.zeros(self.n, dtype=torch.float64, device="cuda")
        on = at[0] == at[1]
        self.diagonal[at[0][on]] = a.values()[on]
        self.a = a.to_sparse_csr()

    def times(self, x):
        return (self.a @ x.unsqueeze(1)).squeeze(1)

    def solve(self, f, tol=1e-13):
        x = torch.zeros_like(f)
        r = f.clone()
        z = r / self.diagonal
        p, rz, stop = z.clone(), torch.dot(r, z), float(f.norm()) * tol
        for k in range(20000):
            q = self.times(p)
            alpha = rz / torch.dot(p, q)
            x += alpha * p
            r -= alpha * q
            if k % 50 == 49 and float(r.norm()) <= stop:
                break
            z = r / self.diagonal
            rz, old = torch.dot(r, z), rz
            p = z + (rz / old) * p
        return x

    def element_products(self, u, w):
        pad = lambda v: torch.cat([v, v.new_zeros(1)])[self.dof]  # noqa: E731  (number -1: a fixed vertex, 0)
        return (pad(u).unsqueeze(2) * self.k1 * pad(w).unsqueeze(1)).sum((1, 2))


def exact(case, seed):
    kind = case["kind"]
    if kind == "batch":
        meshes = list(_batch_meshes(case, seed))
        rhs = case["rhs"]
        sizes = [int((~fixed).sum()) for _, _, fixed in meshes]
        r = np.random.default_rng([int(seed), 2, case["meshes"]])
        f = torch.from_numpy(r.uniform(-1.0, 1.0, sum(sizes) * rhs)).cuda()
        # all meshes as one: block by block, one solve for each right-hand side
        at = np.cumsum([0] + [len(p) for p, _, _ in meshes])
        whole = _Plain(np.concatenate([p for p, _, _ in meshes]),
                       np.concatenate([e + o for (_, e, _), o in zip(meshes, at)]),
                       np.concatenate([fixed for _, _, fixed in meshes]),
                       np.ones(sum(len(e) for _, e, _ in meshes)))
        parts = [b.reshape(rhs, n) for b, n in zip(f.split([n * rhs for n in sizes]), sizes)]
        u = [whole.solve(torch.cat([b[q] for b in parts])).split(sizes) for q in range(rhs)]
        return [torch.cat([torch.cat([u[q][i] for q in range(rhs)]) for i in range(len(sizes))]), None]
    p, e, fixed, m, f, _ = _problem(case, seed)
    plain = _Plain(p, e, fixed, np.exp(m))
    f = torch.from_numpy(f).cuda()
    if kind == "krylov":
        return None  # B_co r is defined by the hierarchy; only a solve says whether it is right
    u = plain.solve(f)
    if kind == "gradient":
        r = np.random.default_rng([int(seed), 3, case["n"]])
        seen = torch.from_numpy(1e-3 * r.standard_normal(plain.n)).cuda()
        w = plain.solve(u - seen)
        return [u, -plain.kappa * plain.element_products(u, w)]
    return [u.cpu().numpy() if kind == "oneshot" or case["host"] else u, None]
