"""The kernels of the solve phase at the sizes where their splits change, against
FP64 reference sums and the CPU oracle.  A sum of k products formed in any order
differs from the exact one by at most k eps sum |a||b|: the tolerances are twice
that (both sides round)."""
import numpy as np
import pytest
import scipy.sparse as sp

import inputs
from oracle import sa as osa
from oracle import solve as osolve

pytestmark = pytest.mark.gpu

torch = pytest.importorskip("torch")

EPS = 2.0 ** -52


def cuda(x):
    return torch.tensor(np.ascontiguousarray(x), dtype=torch.float64, device="cuda")


def arrays(m):
    m = m.tocsr()
    m.sort_indices()
    return m.indptr.astype(np.int32), m.indices.astype(np.int32), m.data.astype(np.float64)


def chain(n):
    """tridiagonal, symmetric positive definite, no two rows alike"""
    d = 2.0 + 1e-4 * (2.0 + np.cos(np.arange(n)))  # coarsens below 64 rows at n = 70001
    return sp.diags([-np.ones(n - 1), d, -np.ones(n - 1)], [-1, 0, 1], shape=(n, n))


def solver(A, M, mask=None, **opts):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_11533_amd as amg
    return amg.HessianSolver(arrays(A), arrays(M), mask, **opts)


# one column and up to four run on vector ALUs (a wavefront per row), more on
# the matrix cores (1, 2, 4, 8 or 16 rows per workgroup and one, two, three, four or
# eight chunks of loads per wavefront at these sizes)
@pytest.mark.parametrize("nb", [1, 2, 3, 4, 7, 16])
@pytest.mark.parametrize("n", [2, 15, 17, 64, 257, 600, 1000, 1030, 2049])
def test_dense_inverse_apply(n, nb):
    g = solver(chain(n), chain(n), nb_max=nb, inner_precision=32, max_coarse=n, dense_max=4096)
    assert g.levels()[0] == 1
    inv = g.dense(0)
    b = np.random.default_rng(n + nb).standard_normal((n, nb))
    mag = np.abs(inv) @ np.abs(b)
    x = g.vcycle_apply(cuda(b), prec=64).cpu().numpy()
    assert (np.abs(x - inv @ b) <= 2 * n * EPS * mag).all()
    i32, b32 = inv.astype(np.float32).astype(np.float64), b.astype(np.float32).astype(np.float64)
    x = g.vcycle_apply(cuda(b), prec=32).cpu().numpy()
    assert (np.abs(x - i32 @ b32) <= 2.0 ** -23 * np.abs(i32 @ b32) + 2 * n * EPS * mag).all()


def banded(n, lens, spread, seed):
    """symmetric, rows of about lens[i % len(lens)] entries within `spread` of the diagonal"""
    rng = np.random.default_rng(seed)
    k = np.resize(lens, n)
    i = np.repeat(np.arange(n), k)
    j = np.clip(i + rng.integers(-spread, spread + 1, len(i)), 0, n - 1)
    m = sp.coo_matrix((rng.standard_normal(len(i)) * 0.01, (i, j)), shape=(n, n)).tocsr()
    if n > 65536:  # a wide, regular coupling as well: i and n - 1 - i
        m = m + sp.coo_matrix((np.full(n, 0.01), (np.arange(n), np.arange(n)[::-1])), shape=(n, n))
    return (m + m.T + 10.0 * sp.eye(n)).tocsr()


# rows of near-equal length (the sliced-ELL copy for every batch), of at most
# eight and of more entries; a few long rows (padding beyond half as many again:
# batches on CSR); offsets beyond 16 bits (CSR throughout)
@pytest.mark.parametrize("nb", [1, 2, 3, 4, 8, 13, 16])
@pytest.mark.parametrize("n,lens,spread", [(3, [1], 1), (63, [2], 9), (65, [3], 20), (1000, [2], 300),
                                           (5000, [9], 900), (3001, [1] * 40 + [70], 1200), (70001, [2], 3)])
def test_products_and_dots(n, lens, spread, nb):
    M = banded(n, lens, spread, n)
    mask = (np.random.default_rng(n).random(n) < 0.02).astype(np.uint8)
    mask[: 2] = [1, 0]
    g = solver(chain(n), M, mask, nb_max=nb, max_coarse=64)
    x = np.random.default_rng(nb).standard_normal((n, nb))
    k = np.diff(M.indptr).max() + 2
    D = sp.diags(1.0 - mask)
    for which, op in enumerate([M, D @ M @ D, D @ M, M @ D]):
        y = g.mass_apply(cuda(x), which).cpu().numpy()
        assert (np.abs(y - op @ x) <= 2 * k * EPS * (abs(op) @ np.abs(x)) + 1e-300).all(), which
        if which < 2:
            q = g.mass_quad(cuda(x), which).numpy()
            ref = np.einsum("ic,ic->c", x, op @ x)
            mag = np.einsum("ic,ic->c", np.abs(x), abs(op) @ np.abs(x))
            assert (np.abs(q - ref) <= 2 * (n + k) * EPS * mag).all(), which


# level-1 matrices of long rows beyond 10 MB in both precisions (six and eight
# entries per lane), more than 65536 level-1 nodes, level-0 launches that sweep more
# rows than they have workgroups; columns about the row's place (16 bits) in the
# natural numbering, anywhere (32 bits) in a random one
@pytest.fixture(scope="module", params=["natural", "shuffled"])
def big(request):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_11533_amd as amg
    p = inputs.config("c3", n=96)
    coords, elems, bc = p.mesh.coords, p.mesh.elems, p.dirichlet
    if request.param == "shuffled":
        perm = np.random.default_rng(96).permutation(p.mesh.nverts)
        inv = np.empty_like(perm)
        inv[perm] = np.arange(len(perm))
        coords, elems, bc = np.ascontiguousarray(coords[perm]), inv[elems].astype(elems.dtype), bc[perm].copy()
    rp, ci, va, vm = amg.assemble_p1(coords, elems, p.kappa)
    gs = {nb: amg.HessianSolver((rp, ci, va), (rp, ci, vm), bc, beta=p.beta, nb_max=nb, inner_precision=32,
                                smoother=1) for nb in (1, 16)}
    n1, nnz1, _, _ = gs[1].level_size(1)
    assert n1 > 65536 and nnz1 > 16 * n1 and 8 * nnz1 >= 1e7
    return gs


@pytest.mark.parametrize("nb", [1, 16])
@pytest.mark.parametrize("level", [0, 1])
def test_large_products(big, level, nb):
    g = big[nb]
    n = g.level_n(level)
    rp, ci, v = g.csr(level, 3)
    M = sp.csr_matrix((v, ci, rp), shape=(n, n))
    x = np.random.default_rng(level).standard_normal((n, nb))
    k = np.diff(rp).max() + 2
    y = g.mass_apply(cuda(x), 0, level=level).cpu().numpy()
    assert (np.abs(y - M @ x) <= 2 * k * EPS * (abs(M) @ np.abs(x))).all()
    if level == 0:
        q = g.mass_quad(cuda(x), 0).numpy()
        # partial sums of at most 2^11 rows per lane, then a tree
        mag = np.einsum("ic,ic->c", np.abs(x), abs(M) @ np.abs(x))
        assert (np.abs(q - np.einsum("ic,ic->c", x, M @ x)) <= 2 * (4096 + k) * EPS * mag).all()


@pytest.mark.parametrize("level", [0, 1])
def test_large_cycles(big, level):
    # a batch's columns are the single columns' cycles; the float32 cycle agrees
    # with the FP64 one to float32 accuracy (1e-4, the bound of the small meshes'
    # test against the oracle)
    n = big[1].level_n(level)
    B = np.random.default_rng(3).standard_normal((n, 16))
    X64 = big[16].vcycle_apply(cuda(B), level=level, prec=64).cpu().numpy()
    X32 = big[16].vcycle_apply(cuda(B), level=level, prec=32).cpu().numpy()
    assert np.linalg.norm(X32 - X64) < 1e-4 * np.linalg.norm(X64)
    for c in (0, 15):
        x = big[1].vcycle_apply(cuda(B[:, c]), level=level, prec=64).cpu().numpy()
        assert np.linalg.norm(x - X64[:, c]) < 1e-13 * np.linalg.norm(x)
        x = big[1].vcycle_apply(cuda(B[:, c]), level=level, prec=32).cpu().numpy()
        assert np.linalg.norm(x - X64[:, c]) < 1e-4 * np.linalg.norm(x)


# the convergence test that runs ahead of the preconditioner ends a CG in the
# iteration in which the textbook loop ends (one apart where rounding decides)
@pytest.mark.parametrize("rtol", [0.5, 1e-3, 1e-7, 1e-12])
@pytest.mark.parametrize("nb", [1, 3])
def test_iterations_to_convergence(rtol, nb):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_11533_amd as amg
    p = inputs.config("c3", n=14)
    rp, ci, va, vm = amg.assemble_p1(p.mesh.coords, p.mesh.elems, p.kappa)
    g = amg.HessianSolver((rp, ci, va), (rp, ci, vm), p.dirichlet, beta=p.beta, nb_max=nb, inner_rtol=rtol,
                          max_coarse=40, dense_solve_max=0)
    h, _, _ = osolve.build_problem(p, osa.Opts(beta=p.beta, inner_rtol=rtol, max_coarse=40, dense_solve_max=0))
    u = np.random.default_rng(9).standard_normal((p.mesh.nverts, nb))
    if nb == 3:
        u[:, 1] = 0.0
    for _ in range(2):  # the second solve expects what the first one took
        y = g.state_solve(cuda(u)).cpu().numpy()
        most = 0
        for c in range(nb):
            o = osolve.Oracle(h)
            ref = o.state_solve(0, u[:, c])
            most = max(most, o.cnt.inner_iters)
            if not u[:, c].any():
                assert not y[:, c].any()
            else:  # two iterates within rtol of the solution in the residual norm
                assert np.linalg.norm(y[:, c] - ref) <= max(100 * rtol, 1e-10) * np.linalg.norm(ref)
        assert abs(g.last_info["inner_iters_max"] - most) <= 1


# vectors without padding columns are read and written where the caller has
# them: any 8-byte alignment, and outputs that overlap the input
@pytest.mark.parametrize("nb", [1, 2, 4])
@pytest.mark.parametrize("shift", [0, 1, 700])
def test_unaligned_and_overlapping_vectors(nb, shift):
    from paper_2001_11533_amd._lib import check, lib
    n = 1501
    M = banded(n, [4], 90, 5)
    g = solver(chain(n), M, nb_max=nb, max_coarse=64, mass_rtol=1e-13)
    x = np.random.default_rng(1).standard_normal((n, nb))
    aligned = cuda(x)
    for off in (0, 1):
        buf = torch.zeros(2 * n * nb + 8, dtype=torch.float64, device="cuda")
        for out in (off + shift, off + shift + n * nb // 2):
            buf[off:off + n * nb] = aligned.reshape(-1)
            check(lib().amg_mass_apply(g._h, 0, 0, buf.data_ptr() + 8 * off, buf.data_ptr() + 8 * out, nb), g._h)
            assert torch.equal(buf[out:out + n * nb].reshape(n, nb), g.mass_apply(aligned))
        buf[off:off + n * nb] = aligned.reshape(-1)
        z = buf[off:off + n * nb].reshape(n, nb)
        for f in (g.state_solve, g.adjoint_solve, g.hessian_apply, g.vcycle_apply):
            a, b = f(z), f(aligned)
            assert torch.linalg.norm(a - b) <= 1e-12 * torch.linalg.norm(b), f
            assert torch.equal(z, aligned)


def stencil(n, offs, seed):
    """symmetric, the diagonals 0, +-offs with every tenth entry missing: rows of unequal
    length, in slices of 64 that pad by little"""
    rng = np.random.default_rng(seed)
    m = sp.diags([np.where(rng.random(max(n - o, 0)) < 0.9, rng.uniform(0.5, 1.0, max(n - o, 0)), 0.0) for o in offs],
                 list(offs), shape=(n, n)).tocsr()
    m.eliminate_zeros()
    return (m + m.T + 40.0 * sp.eye(n)).tocsr()


def padding(M):
    """entries of the sliced-ELL copy over stored entries"""
    k = np.diff(M.indptr)
    return sum(64 * k[s:s + 64].max() for s in range(0, len(k), 64)) / M.nnz


# a value that is not finite reaches the rows that hold its node and no others,
# whatever entries a matrix copy pads its rows with: single values at the smallest
# column of a slice of 64 rows.  Rows of at most eight and of more entries, on CSR and
# (one column always, batches from 2^15 lanes or 2^16 long rows on) in sliced ELL; a
# few long rows, on CSR for batches
@pytest.mark.parametrize("nb", [1, 2, 3, 4, 8, 16])
@pytest.mark.parametrize("bad", [np.inf, -np.inf, np.nan])
@pytest.mark.parametrize("n,offs", [(64, (1, 5, 9)), (127, (1, 5, 9)), (1000, (1, 30, 31)), (5000, range(1, 9)),
                                    (3001, None), (33001, (1, 30, 31)), (65601, range(1, 9))])
def test_products_keep_non_finite_values_to_their_rows(n, offs, bad, nb):
    if offs:
        M = stencil(n, offs, n)
        assert padding(M) <= 1.5
    else:
        M = banded(n, [1] * 40 + [70], 1200, n)
        assert padding(M) > 1.5
    M.sort_indices()
    g = solver(chain(n), M, nb_max=nb, max_coarse=64)
    x = np.random.default_rng(nb).standard_normal((n, nb))
    x0, hit = x.copy(), np.zeros((n, nb), dtype=bool)
    for sl, c in ((0, 0), ((n - 1) // 64 // 2, nb - 1)):
        k = M.indices[M.indptr[64 * sl]:M.indptr[min(64 * (sl + 1), n)]].min()
        x[k, c], x0[k, c] = bad, 0.0
        hit[M.indices[M.indptr[k]:M.indptr[k + 1]], c] = True  # M is symmetric: row k holds the column's rows
    y = g.mass_apply(cuda(x)).cpu().numpy()
    assert (np.isnan(y[hit]) if np.isnan(bad) else ~np.isfinite(y[hit])).all()
    k = np.diff(M.indptr).max() + 2
    err = np.abs(np.where(hit, 0.0, y - M @ x0))
    assert (err <= 2 * k * EPS * (abs(M) @ np.abs(x0))).all()


# ... and an infinity in a dense solve's right-hand side, where every product with it
# is infinite (a tridiagonal M-matrix has a positive inverse), leaves infinities
@pytest.mark.parametrize("nb", [1, 4, 7, 16])
@pytest.mark.parametrize("n", [15, 64, 257, 600])
@pytest.mark.parametrize("prec", [32, 64])
def test_dense_apply_of_infinities(n, nb, prec):
    g = solver(chain(n), chain(n), nb_max=nb, inner_precision=32, max_coarse=n, dense_max=4096)
    inv = g.dense(0).astype(np.float32 if prec == 32 else np.float64).astype(np.float64)
    assert (inv > 0).all()
    for k in (0, n - 2, n - 1):
        b = np.random.default_rng(n + nb).standard_normal((n, nb))
        b[k, 0] = np.inf
        x = g.vcycle_apply(cuda(b), prec=prec).cpu().numpy()
        assert (x[:, 0] == np.inf).all()
        assert np.isfinite(x[:, 1:]).all()


# an inner solve that does not converge leaves the output as it was
@pytest.mark.parametrize("nb", [1, 2, 3, 4])
@pytest.mark.parametrize("mode", [{}, {"inner_precision": 32}, {"inner_precision": 32, "mixed_mode": 1}])
def test_outputs_after_a_failed_inner_solve(nb, mode):
    from paper_2001_11533_amd._lib import lib
    n = 1501
    g = solver(chain(n), banded(n, [4], 90, 5), nb_max=nb, max_coarse=64, dense_solve_max=0, inner_maxit=1, **mode)
    x = cuda(np.random.default_rng(1).standard_normal((n, nb)))
    y = torch.full_like(x, -7.0)
    for f in (lib().state_solve, lib().adjoint_solve, lib().hessian_apply):
        assert f(g._h, 0, x.data_ptr(), y.data_ptr(), nb, None) == -4
        torch.cuda.synchronize()
        assert bool((y == -7.0).all())


# every mass product and its dots on matrices that pad by little: around the rows from
# which a batch runs on the sliced-ELL copy (2^13, 2^14 and 2^15 at 16, 8 and up to four
# columns; 2^16 where rows are longer than eight entries), one slice, ragged last
# slices, one and several rounds of eight entries per lane
@pytest.mark.parametrize("nb", [1, 2, 3, 4, 8, 13, 16])
@pytest.mark.parametrize("n,offs", [(64, (1, 5, 9)), (127, (1, 5, 9)), (1000, (1, 30, 31)), (5000, range(1, 9)),
                                    (8191, (1, 30, 31)), (8193, (1, 30, 31)), (16385, (1, 30, 31)),
                                    (32769, (1, 30, 31)), (65535, range(1, 9)), (65601, range(1, 9))])
def test_products_and_dots_on_sliced_ell(n, offs, nb):
    M = stencil(n, offs, n)
    assert padding(M) <= 1.5
    mask = (np.random.default_rng(n).random(n) < 0.02).astype(np.uint8)
    mask[: 2] = [1, 0]
    g = solver(chain(n), M, mask, nb_max=nb, max_coarse=64)
    x = np.random.default_rng(nb).standard_normal((n, nb))
    k = np.diff(M.indptr).max() + 2
    D = sp.diags(1.0 - mask)
    for which, op in enumerate([M, D @ M @ D, D @ M, M @ D]):
        y = g.mass_apply(cuda(x), which).cpu().numpy()
        assert (np.abs(y - op @ x) <= 2 * k * EPS * (abs(op) @ np.abs(x))).all(), which
        if which < 2:
            q = g.mass_quad(cuda(x), which).numpy()
            mag = np.einsum("ic,ic->c", np.abs(x), abs(op) @ np.abs(x))
            assert (np.abs(q - np.einsum("ic,ic->c", x, op @ x)) <= 2 * (n + k) * EPS * mag).all(), which


# the convergence test ahead of the preconditioner changes neither iterates nor counts:
# the same solves with captured graphs, which run without it.  One and two columns
# fold their finalize into the next product here, eight and sixteen do not.
@pytest.mark.parametrize("n,nb", [(14, 1), (14, 2), (32, 8), (24, 16)])
@pytest.mark.parametrize("mode", [{}, {"inner_precision": 32}, {"inner_precision": 32, "mixed_mode": 1}])
@pytest.mark.parametrize("rtol", [1e-2, 1e-9])
def test_early_convergence_test_is_invisible(n, nb, mode, rtol):
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2001_11533_amd as amg
    p = inputs.config("c3", n=n)
    rp, ci, va, vm = amg.assemble_p1(p.mesh.coords, p.mesh.elems, p.kappa)
    rng = np.random.default_rng(n)
    x, y, z = (p.mesh.coords * np.pi).T
    u = np.stack([rng.standard_normal(len(x)) if c % 2 else np.sin(x * (c + 1)) * np.sin(y) * np.sin(z)
                  for c in range(nb)], axis=1)  # smooth and rough columns stop in different iterations
    if nb > 2:
        u[:, 2] = 0.0
    got = []
    for graphs in (1, 0, 2):
        g = amg.HessianSolver((rp, ci, va), (rp, ci, vm), p.dirichlet, beta=p.beta, nb_max=nb, inner_rtol=rtol,
                              max_coarse=40, dense_solve_max=0, use_graphs=graphs, **mode)
        r = []
        for v in (u, u[:, ::-1].copy(), u):  # later solves expect what the ones before took
            y = g.state_solve(cuda(v))
            r.append((y, g.last_info["inner_iters_total"], g.last_info["inner_iters_max"]))
        got.append(r)
    for other in got[1:]:
        for (a, ia, ma), (b, ib, mb) in zip(got[0], other):
            assert (ia, ma) == (ib, mb)
            assert torch.equal(a, b)
