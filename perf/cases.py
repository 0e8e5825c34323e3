"""The work a user of this package has it do, as measurable cases.

A program of this package assembles P1 matrices of a simplicial mesh, builds a
HessianSolver on them and then asks it for state and adjoint solves, Hessian
actions, gradients of the reduced functional or whole reduced solves, for one
desired state or a batch of them.  The cases below take these calls over the
range of meshes of the package's workloads: 2D squares (n x n cells, two
triangles each) and 3D cubes (n^3 cells, six Kuhn tetrahedra each), uniform,
jittered or renumbered, with constant, checkerboard, log-normal or ball
coefficients, Dirichlet nodes on the whole boundary or on one face.
"""
import itertools
import math

import numpy as np
import torch

import paper_2001_11533_amd as amg

DEV = "cuda"


def listed():
    return [
        # the smallest call: one mass product on the 32^2 mesh, as an outer optimiser's
        # inner products and norms make many of; launches and host work are all of it
        {"name": "mass_2d_32", "op": "mass", "dim": 2, "n": 32, "kappa": "const"},
        # the smallest whole solve: the paper's 2D model problem, default options
        {"name": "solve_2d_32", "op": "solve", "dim": 2, "n": 32, "kappa": "const"},
        # one step of a gradient method for 8 controls at once through torch.autograd:
        # a state solve forward, an adjoint solve backward, FP64 throughout
        {"name": "gradient_2d_256x8", "op": "gradient", "dim": 2, "n": 256, "kappa": "checker", "jitter": 0.2,
         "nb": 8},
        # the ordinary 2D solve on an irregular mesh with a high-contrast coefficient
        # and weak regularisation, FP64 throughout, default options
        {"name": "solve_2d_256", "op": "solve", "dim": 2, "n": 256, "kappa": "checker", "jitter": 0.2,
         "beta": 1e-4},
        # new coefficient on the benchmark's mesh: both matrices assembled on the GPU
        {"name": "assemble_3d_64", "op": "assemble", "dim": 3, "n": 64, "kappa": "lognormal"},
        # the benchmark's step: setup and reduced solve at 64^3, float32 V-cycles with
        # Chebyshev smoothing inside FP64 CG
        {"name": "step_3d_64", "op": "step", "dim": 3, "n": 64, "kappa": "lognormal", "beta": 1e-3,
         "precision": 32, "smoother": 1},
        # one Hessian action of a user's own Krylov method, FP64 with the default smoother
        {"name": "hessian_3d_64", "op": "hessian", "dim": 3, "n": 64, "kappa": "lognormal", "beta": 1e-3},
        # setup and one state solve on a mesh whose vertices are numbered at random, as
        # meshes from a generator are; ball coefficient, Dirichlet nodes on one face
        {"name": "setup_3d_48_shuffled", "op": "setup", "dim": 3, "n": 48, "kappa": "ball", "shuffle": True,
         "face": True},
        # an odd batch on an odd mesh: 5 adjoint solves at 37^3, float32 V-cycles
        {"name": "adjoint_3d_37x5", "op": "adjoint", "dim": 3, "n": 37, "kappa": "lognormal", "nb": 5,
         "precision": 32, "smoother": 1},
        # the benchmark's batch: 16 desired states in one reduced solve
        {"name": "solve_3d_64x16", "op": "solve", "dim": 3, "n": 64, "kappa": "lognormal", "beta": 1e-3, "nb": 16,
         "precision": 32, "smoother": 1},
        # the widest batch on the largest mesh: 16 states at 128^3
        {"name": "state_3d_128x16", "op": "state", "dim": 3, "n": 128, "kappa": "lognormal", "var": 2.0, "nb": 16,
         "precision": 32, "smoother": 1},
        # the largest single problem, setup and solve: two Hessian levels, as the
        # benchmark runs it at this beta
        {"name": "step_3d_128", "op": "step", "dim": 3, "n": 128, "kappa": "lognormal", "var": 2.0, "beta": 1e-4,
         "precision": 32, "smoother": 1, "levels": 2},
    ]


def draw(rng):
    op = rng.choice(["mass", "state", "adjoint", "hessian", "gradient", "solve", "solve", "setup", "step", "assemble"])
    dim = rng.choice([2, 3, 3])
    lo, hi = (24, 400) if dim == 2 else (10, 128 if op in ("assemble", "mass", "state") else 90)
    n = int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))
    c = {"op": op, "dim": dim, "n": n}
    c["kappa"] = rng.choice(["const", "checker", "lognormal"] if dim == 2 else ["lognormal", "lognormal", "ball"])
    if dim == 2 and rng.random() < 0.5:
        c["jitter"] = 0.2
    if dim == 3 and n <= 64 and rng.random() < 0.25:
        c["shuffle"] = True
    if c["kappa"] == "ball":
        c["face"] = True
    if op != "assemble":
        c["precision"] = rng.choice([32, 64])
        c["smoother"] = rng.choice([0, 1])
        c["beta"] = rng.choice([1e-1, 1e-2, 1e-2, 3e-3])
        c["nb"] = rng.choice([1, 1, 1, 2, 3, 5, 8, 11, 16] if n ** dim <= 300_000 else [1, 1, 1, 2, 3])
    return c


# ---------------------------------------------------------------- inputs

def _grid(dim, n):
    """(N, dim) integer lattice points, the first coordinate running fastest."""
    ax = torch.arange(n + 1, device=DEV)
    return torch.stack([g.reshape(-1) for g in torch.meshgrid(*[ax] * dim, indexing="ij")][::-1], dim=1)


def _mesh(case, rng):
    """Coordinates, elements and Dirichlet flags of the case's mesh, on the GPU."""
    dim, n = case["dim"], case["n"]
    p = _grid(dim, n)
    coords = p.double() / n
    step = torch.tensor([(n + 1) ** a for a in range(dim)], device=DEV)
    base = (_grid(dim, n - 1) * step).sum(1)
    cells = []
    for perm in itertools.permutations(range(dim)):
        v = [base]
        for a in perm:
            v.append(v[-1] + step[a])
        if dim == 2 and perm == (1, 0):
            v = [v[0], v[2], v[1]]  # counter-clockwise
        cells.append(torch.stack(v, dim=1))
    elems = torch.stack(cells, dim=1).reshape(-1, dim + 1)
    edge = ((p == 0) | (p == n)).any(1)
    if case.get("jitter"):
        d = torch.from_numpy(rng.uniform(-1.0, 1.0, size=(p.shape[0], dim))).to(DEV) * (case["jitter"] / n)
        coords = torch.where(edge[:, None], coords, coords + d)
    mask = p[:, -1] == 0 if case.get("face") else edge
    if case.get("shuffle"):
        perm = torch.from_numpy(rng.permutation(p.shape[0])).to(DEV)  # old vertex -> new vertex
        inv = torch.argsort(perm)
        coords, mask, elems = coords[inv], mask[inv], perm[elems]
    return coords.contiguous(), elems.to(torch.int32).contiguous(), mask.to(torch.uint8).contiguous()


def _kappa(case, rng, coords, elems):
    """One diffusion coefficient per element, at its centroid."""
    dim = case["dim"]
    c = sum(coords[elems[:, a].long()] for a in range(dim + 1)) / (dim + 1)
    if case["kappa"] == "const":
        return torch.ones_like(c[:, 0])
    if case["kappa"] == "checker":
        q = (4 * c).floor().long().clamp(max=3).sum(1)
        return torch.where(q % 2 == 0, 1.0, 1e3).double()
    if case["kappa"] == "ball":
        return torch.where((c - 0.5).norm(dim=1) <= 0.25, float(rng.uniform(0.05, 0.2)), 1.0).double()
    var, modes = case.get("var", 1.0), 16
    w = rng.integers(-4, 5, size=(modes, dim))
    w[(w == 0).all(1), 0] = 1
    phi = rng.uniform(0.0, 2.0 * math.pi, size=modes)
    g = torch.zeros_like(c[:, 0])
    for m in range(modes):
        g += torch.cos(2.0 * math.pi * (c @ torch.tensor(w[m], dtype=torch.float64, device=DEV)) + float(phi[m]))
    return torch.exp(g * math.sqrt(2.0 * var / modes))


def _bumps(rng, coords, nb):
    """nb desired states, each a sum of eight Gaussian bumps."""
    out = torch.zeros((coords.shape[0], nb), dtype=torch.float64, device=DEV)
    for k in range(nb):
        for a, x in zip(rng.uniform(0.0, 1.0, 8), rng.uniform(0.0, 1.0, (8, coords.shape[1]))):
            r2 = ((coords - torch.from_numpy(x).to(DEV)) ** 2).sum(1)
            out[:, k] += float(a) * torch.exp(-r2 / (2 * 0.05 ** 2))
    return out


def _inputs(case, seed):
    rng = np.random.default_rng(seed)
    coords, elems, mask = _mesh(case, rng)
    kappa = _kappa(case, rng, coords, elems)
    if case["kappa"] == "const":  # no other input of an assembly depends on the seed
        kappa *= float(rng.uniform(0.5, 2.0))
    nb = case.get("nb", 1)
    v = {}
    if case["op"] in ("solve", "step", "gradient"):
        v["yd"] = _bumps(rng, coords, nb)
    if case["op"] not in ("solve", "step", "assemble"):
        gen = torch.Generator(device=DEV).manual_seed(int(rng.integers(1 << 31)))
        v["u"] = torch.randn((coords.shape[0], nb), dtype=torch.float64, device=DEV, generator=gen)
    if nb == 1:  # a single vector is passed as one
        v = {k: x[:, 0].contiguous() for k, x in v.items()}
    return coords, elems, mask, kappa, v


def _options(case):
    return dict(beta=case.get("beta", 1e-2), inner_precision=case.get("precision", 64),
                smoother=case.get("smoother", 0), nb_max=case.get("nb", 1), hess_levels=case.get("levels", 0))


def prepare(case, seed):
    coords, elems, mask, kappa, v = _inputs(case, seed)
    s = {"op": case["op"], "options": _options(case), **v}
    if case["op"] == "assemble":
        return {**s, "mesh": (coords, elems, kappa)}
    rp, ci, va, vm = amg.assemble_p1_device(coords, elems, kappa)
    s["matrices"] = ((rp, ci, va), (rp, ci, vm), mask)
    if case["op"] not in ("setup", "step"):
        s["solver"] = amg.HessianSolver(*s["matrices"], **s["options"])
    return s


def run(state):
    op, solver = state["op"], state.get("solver")
    if op == "assemble":
        return amg.assemble_p1_device(*state["mesh"])
    if op in ("setup", "step"):
        solver = amg.HessianSolver(*state["matrices"], **state["options"])
        out = solver.state_solve(state["u"]) if op == "setup" else solver.reduced_solve(state["yd"])[0]
        solver.close()
        return out
    if op == "mass":
        return solver.mass_apply(state["u"])
    if op == "state":
        return solver.state_solve(state["u"])
    if op == "adjoint":
        return solver.adjoint_solve(state["u"])
    if op == "hessian":
        return solver.hessian_apply(state["u"])
    if op == "gradient":
        u = state["u"].detach().requires_grad_(True)
        J = amg.reduced_functional(u, state["yd"], solver)
        J.sum().backward()
        return {"J": J.detach(), "grad": u.grad}
    return solver.reduced_solve(state["yd"])[0]


# ---------------------------------------------------------------- what a pass cannot do without

def work(case):
    """Each input read once, each output written once; one use of every operator in flops."""
    dim, n, nb, op = case["dim"], case["n"], case.get("nb", 1), case["op"]
    N = (n + 1) ** dim
    if dim == 2:
        ne, edges = 2 * n * n, 2 * n * (n + 1) + n * n
    else:
        ne, edges = 6 * n ** 3, 3 * n * (n + 1) ** 2 + 3 * n * n * (n + 1) + n ** 3
    nnz = N + 2 * edges
    if op == "assemble":
        return {"bytes": 8 * dim * N + (4 * (dim + 1) + 8) * ne + 4 * (N + 1) + 20 * nnz,
                "flops": ne * (dim + 1) ** 2 * (2 * dim + 2)}
    matrix = 12 * nnz + 4 * (N + 1)  # one CSR matrix, FP64
    vectors = {"solve": 2, "step": 2, "gradient": 3, "mass": 2, "state": 2, "adjoint": 2, "hessian": 2, "setup": 2}[op]
    matrices = 1 if op == "mass" else 2
    products = {"mass": 1, "state": 2, "adjoint": 2, "setup": 2, "hessian": 5, "gradient": 5, "solve": 5, "step": 5}[op]
    return {"bytes": matrices * matrix + 8 * vectors * N * nb, "flops": 2 * products * nnz * nb}


# ---------------------------------------------------------------- the same results in plain torch, 64 bits

def _assembled(coords, elems, kappa):
    """(rowptr, col, stiffness, mass) with every pair of vertices that share an element stored."""
    e, (N, dim) = elems.long(), coords.shape
    x = [coords[e[:, a]] for a in range(dim + 1)]
    d = [x[a] - x[0] for a in range(1, dim + 1)]
    if dim == 2:
        det = d[0][:, 0] * d[1][:, 1] - d[0][:, 1] * d[1][:, 0]
        g = [torch.stack([d[1][:, 1], -d[1][:, 0]], 1), torch.stack([-d[0][:, 1], d[0][:, 0]], 1)]
    else:
        g = [torch.linalg.cross(d[1], d[2]), torch.linalg.cross(d[2], d[0]), torch.linalg.cross(d[0], d[1])]
        det = (d[0] * g[0]).sum(1)
    g = [v / det[:, None] for v in g]
    g = [-sum(g)] + g
    meas = det.abs() / math.factorial(dim)
    pairs = [(a, b) for a in range(dim + 1) for b in range(dim + 1)]
    key, place = torch.unique(torch.cat([e[:, a] * N + e[:, b] for a, b in pairs]), return_inverse=True)
    place = place.reshape(len(pairs), -1)
    A, M = torch.zeros((2, key.numel()), dtype=torch.float64, device=DEV)
    for k, (a, b) in enumerate(pairs):
        A.index_add_(0, place[k], kappa * meas * (g[a] * g[b]).sum(1))
        M.index_add_(0, place[k], meas * ((2.0 if a == b else 1.0) / ((dim + 1) * (dim + 2))))
    rowptr = torch.searchsorted(key, torch.arange(N + 1, device=DEV) * N)
    return rowptr, key % N, A, M


def _sparse_lines(case, rowptr, col, val):
    """Inverse of a 2D matrix in the natural numbering, block tridiagonal over the mesh lines."""
    m = case["n"] + 1
    row = torch.repeat_interleave(torch.arange(m * m, device=DEV), rowptr[1:] - rowptr[:-1])
    D, E = torch.zeros((2, m, m, m), dtype=torch.float64, device=DEV)  # diagonal blocks, blocks below them
    for B, off in ((D, 0), (E, 1)):
        at = row // m - col // m == off
        B[row[at] // m, row[at] % m, col[at] % m] = val[at]
    D, E = D.cpu(), E.cpu()
    inv = []
    for k in range(m):
        S = D[k] if k == 0 else D[k] - E[k] @ inv[-1] @ E[k].T
        inv.append(torch.linalg.inv((S + S.T) / 2))

    def solve(F):
        f = F.cpu().reshape(m, m, -1)
        z = [f[0]]
        for k in range(1, m):
            z.append(f[k] - E[k] @ (inv[k - 1] @ z[-1]))
        y = [inv[-1] @ z[-1]]
        for k in range(m - 2, -1, -1):
            y.append(inv[k] @ (z[k] - E[k + 1].T @ y[-1]))
        return torch.stack(y[::-1]).reshape(m * m, -1).to(DEV)
    return solve


def _cg(apply, F, dinv, tol, most, every):
    """Conjugate gradients on every column, until all residuals are below tol."""
    x, r = torch.zeros_like(F), F.clone()
    z = r * dinv
    p, rz, stop = z.clone(), (r * z).sum(0), tol * F.norm(dim=0)
    for k in range(most):
        q = apply(p)
        a = rz / (p * q).sum(0).clamp_min(1e-300)
        x.addcmul_(p, a.expand_as(p))
        r.addcmul_(q, a.expand_as(q), value=-1.0)
        if k % every == every - 1 and bool((r.norm(dim=0) <= stop).all()):
            break
        z = r * dinv
        new = (r * z).sum(0)
        p.mul_(new / rz.clamp_min(1e-300)).add_(z)
        rz = new
    return x


def exact(case, seed):
    op, dim = case["op"], case["dim"]
    if op == "step" and case["n"] ** dim > 500_000:
        return None  # some fifty Hessian actions of a thousand iterations each
    coords, elems, mask, kappa, v = _inputs(case, seed)
    rowptr, col, A, M = _assembled(coords, elems, kappa)
    if op == "assemble":
        return rowptr.to(torch.int32), col.to(torch.int32), A, M
    N, beta = coords.shape[0], _options(case)["beta"]
    row = torch.repeat_interleave(torch.arange(N, device=DEV), rowptr[1:] - rowptr[:-1])
    keep = (mask == 0).double()
    A = torch.where(row == col, torch.where(mask[row] > 0, 1.0, A), A * keep[row] * keep[col])
    matA, matM = (torch.sparse_csr_tensor(rowptr, col, x, (N, N)) for x in (A, M))
    K1 = keep[:, None]
    if dim == 2:
        solve = _sparse_lines(case, rowptr, col, A)
    else:
        dinv = 1.0 / A[row == col][:, None]

        def solve(F):
            return _cg(lambda p: matA @ p, F, dinv, 1e-14, 5000, 25)

    def hessian(x):
        t = solve(K1 * (matM @ (K1 * solve(K1 * (matM @ x)))))
        return matM @ (K1 * t + beta * x)

    one = case.get("nb", 1) == 1
    v = {k: x.reshape(N, -1) for k, x in v.items()}
    if op == "mass":
        out = matM @ v["u"]
    elif op in ("state", "setup"):
        out = solve(K1 * (matM @ v["u"]))
    elif op == "adjoint":
        out = matM @ (K1 * solve(v["u"]))
    elif op == "hessian":
        out = hessian(v["u"])
    elif op == "gradient":
        e = solve(K1 * (matM @ v["u"])) - v["yd"]
        w, m = K1 * (matM @ (K1 * e)), matM @ v["u"]
        J = 0.5 * (e * w).sum(0) + 0.5 * beta * (v["u"] * m).sum(0)
        g = matM @ (K1 * solve(w)) + beta * m
        return {"J": J.reshape(()) if one else J, "grad": g.reshape(-1) if one else g}
    else:
        rhs = matM @ (K1 * solve(K1 * (matM @ (K1 * v["yd"]))))
        scale = (beta * M[row == col])[:, None].reciprocal()  # the Hessian is close to beta times the mass matrix
        out = _cg(hessian, rhs, scale, 1e-12, 200, 1)
    return out.reshape(-1) if one else out
