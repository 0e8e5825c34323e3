"""P1 assembly on the GPU (amg_p1_pattern_device / amg_p1_assemble_device)
against the host assembler, bit for bit, and its argument checks.  The host
assembler is itself pinned to the oracle's assembly (tests/test_lib_host.py)."""
import ctypes as C

import numpy as np
import pytest

import inputs

torch = pytest.importorskip("torch")

pytestmark = pytest.mark.gpu


def _need_gpu():
    if not torch.cuda.is_available():
        pytest.skip("no GPU")


def dev(x, dt):
    return torch.as_tensor(np.ascontiguousarray(x)).to(dtype=dt, device="cuda")


def renumbered(m, seed):
    # the same mesh with a random vertex numbering: element lists around a
    # vertex arrive out of order, and rows gather far-apart columns
    rng = np.random.default_rng(seed)
    perm = rng.permutation(m.nverts)
    inv = np.empty_like(perm)
    inv[perm] = np.arange(len(perm))
    return np.ascontiguousarray(m.coords[perm]), inv[m.elems].astype(np.int32)


@pytest.mark.parametrize("kind", ["2d", "2dj", "3d", "3d_renumbered", "3d64"])
def test_device_assembly_bit_identical_to_host(kind):
    _need_gpu()
    import paper_2001_11533_amd as amg
    m = {"2d": lambda: inputs.mesh2d(9), "2dj": lambda: inputs.mesh2d(40, jitter=0.2),
         "3d": lambda: inputs.mesh3d(7), "3d_renumbered": lambda: inputs.mesh3d(9),
         "3d64": lambda: inputs.mesh3d(64)}[kind]()
    kappa = inputs.kappa_lognormal(m, 1.0)
    coords, elems = m.coords, m.elems
    if kind == "3d_renumbered":
        coords, elems = renumbered(m, 7)
    print(f"[assembly] {kind}: nv={len(coords)} ne={len(elems)}", flush=True)
    rp, ci, va, vm = amg.assemble_p1(coords, elems, kappa)
    r2, c2, a2, m2 = amg.assemble_p1_device(dev(coords, torch.float64), dev(elems, torch.int32),
                                            dev(kappa, torch.float64))
    assert np.array_equal(r2.cpu().numpy(), rp)
    assert np.array_equal(c2.cpu().numpy(), ci)
    # the same operations in the same order: equal to the last bit
    assert np.array_equal(a2.cpu().numpy().view(np.int64), va.view(np.int64))
    assert np.array_equal(m2.cpu().numpy().view(np.int64), vm.view(np.int64))


def test_device_assembly_rejects_bad_input():
    _need_gpu()
    import paper_2001_11533_amd as amg
    from paper_2001_11533_amd import AmgError
    from paper_2001_11533_amd._lib import lib
    m = inputs.mesh2d(6)
    kappa = inputs.kappa_lognormal(m, 1.0)
    coords, elems, kap = dev(m.coords, torch.float64), dev(m.elems, torch.int32), dev(kappa, torch.float64)
    bad = elems.clone()
    bad[3, 1] = m.nverts                       # vertex id out of range
    with pytest.raises(AmgError) as e:
        amg.assemble_p1_device(coords, bad, kap)
    assert e.value.code == -1
    bad[3, 1] = -1
    with pytest.raises(AmgError) as e:
        amg.assemble_p1_device(coords, bad, kap)
    assert e.value.code == -1
    # an nnz that is not the mesh graph's is refused before anything is written
    rp, ci, va, vm = amg.assemble_p1_device(coords, elems, kap)
    nnz = int(ci.numel())
    col = torch.full((nnz,), -7, dtype=torch.int32, device="cuda")
    L = lib()
    rc = L.amg_p1_assemble_device(2, m.nverts, coords.data_ptr(), len(m.elems), elems.data_ptr(), kap.data_ptr(),
                                  nnz - 1, rp.data_ptr(), col.data_ptr(), va.data_ptr(), vm.data_ptr(), None)
    assert rc == -1
    assert bool((col == -7).all())
    n = C.c_int32(0)
    assert L.amg_p1_pattern_device(4, m.nverts, len(m.elems), elems.data_ptr(), C.byref(n), None) == -1
    assert L.amg_p1_pattern_device(2, m.nverts, len(m.elems), None, C.byref(n), None) == -1


def ring_mesh(dim, k, degenerate=False):
    # k simplices around one vertex (2D) or one edge (3D), whose rows then have k
    # elements and k + 1 or k + 2 entries, on vertices numbered at random
    rng = np.random.default_rng(100 * dim + k)
    t = 2.0 * np.pi * np.arange(k) / k
    ring = np.stack([np.cos(t), np.sin(t)] + [0.1 * np.sin(3 * t)] * (dim - 2), axis=1)
    hub = np.zeros((1, 2)) if dim == 2 else np.array([[0.0, 0.0, -1.0], [0.0, 0.0, 1.0]])
    h = len(hub)
    nxt = (np.arange(k) + 1) % k
    elems = np.stack([np.full(k, a) for a in range(h)] + [h + np.arange(k), h + nxt], axis=1)
    if degenerate:  # an element that holds a vertex twice
        elems[k // 2, -1] = elems[k // 2, -2]
    perm = rng.permutation(h + k)
    coords = np.empty((h + k, dim))
    coords[perm] = np.concatenate([hub, ring]) + 0.01 * rng.standard_normal((h + k, dim))
    return coords, perm[elems[rng.permutation(k)]].astype(np.int32), rng.uniform(0.5, 2.0, k)


# around the limits of the row kernels: 32 and 64 elements per row, 127 entries
@pytest.mark.parametrize("dim", [2, 3])
@pytest.mark.parametrize("k", [3, 31, 32, 33, 63, 64, 65, 124, 125, 126, 127, 128, 300])
@pytest.mark.parametrize("degenerate", [False, True])
def test_rows_at_the_limits_of_the_row_kernels(dim, k, degenerate):
    _need_gpu()
    import paper_2001_11533_amd as amg
    print(f"[assembly] ring dim={dim} k={k} degenerate={degenerate}", flush=True)
    coords, elems, kappa = ring_mesh(dim, k, degenerate)
    with np.errstate(all="ignore"):
        ref = amg.assemble_p1(coords, elems, kappa)
    got = [x.cpu().numpy() for x in amg.assemble_p1_device(dev(coords, torch.float64), dev(elems, torch.int32),
                                                           dev(kappa, torch.float64))]
    for a, b in zip(got, ref):
        assert np.array_equal(a, b, equal_nan=a.dtype == np.float64)


# a plan serves any number of fills: new coordinates and coefficients, then the first
# ones again, each against the host assembler; the ring's hub has more elements than
# the row kernels hold, so its fills also sort the plan's lists
@pytest.mark.parametrize("kind", ["2d", "3d", "ring2", "ring3", "loose"])
def test_a_plan_fills_repeatedly(kind):
    _need_gpu()
    import paper_2001_11533_amd as amg
    from paper_2001_11533_amd._lib import check, lib
    L = lib()
    if kind.startswith("ring"):
        coords, elems, kappa = ring_mesh(int(kind[4]), 100)
    else:
        m = inputs.mesh2d(9) if kind == "2d" else inputs.mesh3d(5)
        coords, elems, kappa = m.coords, m.elems.astype(np.int32), inputs.kappa_lognormal(m, 1.0)
    if kind == "loose":  # vertices of no element
        coords = np.concatenate([coords, np.ones((3, 3))])
    dim, nv, ne = coords.shape[1], len(coords), len(elems)
    print(f"[assembly] plan {kind}: nv={nv} ne={ne}", flush=True)
    rng = np.random.default_rng(1)
    fills = [(coords, kappa), (coords + 0.01 * rng.standard_normal(coords.shape), rng.uniform(0.5, 2.0, ne)),
             (coords, kappa)]
    e = dev(elems, torch.int32)
    plan, nnz = C.c_void_p(), C.c_int32(0)
    check(L.amg_p1_plan_device(dim, nv, ne, e.data_ptr(), C.byref(nnz), None, C.byref(plan)))
    for xy, k in fills:
        ref = amg.assemble_p1(xy, elems, k)
        assert nnz.value == len(ref[1])
        x, kd = dev(xy, torch.float64), dev(k, torch.float64)
        out = [torch.full((nv + 1,), -7, dtype=torch.int32, device="cuda"),
               torch.full((nnz.value,), -7, dtype=torch.int32, device="cuda"),
               torch.full((nnz.value,), -7.0, dtype=torch.float64, device="cuda"),
               torch.full((nnz.value,), -7.0, dtype=torch.float64, device="cuda")]
        torch.cuda.synchronize()
        check(L.amg_p1_assemble_planned(plan, x.data_ptr(), e.data_ptr(), kd.data_ptr(), *[o.data_ptr() for o in out]))
        for a, b in zip(out, ref):
            assert np.array_equal(a.cpu().numpy(), b)
    assert L.amg_p1_plan_destroy(plan) == 0


def test_plan_errors():
    _need_gpu()
    from paper_2001_11533_amd._lib import lib
    L = lib()
    m = inputs.mesh2d(6)
    e = dev(m.elems, torch.int32)
    n = C.c_int32(0)

    def make(dim=2, nv=m.nverts, ne=len(m.elems), elems=e, nnz=n):
        plan = C.c_void_p(1234)
        rc = L.amg_p1_plan_device(dim, nv, ne, None if elems is None else elems.data_ptr(),
                                  None if nnz is None else C.byref(nnz), None, C.byref(plan))
        return rc, plan

    for kw in ({"dim": 4}, {"nv": 0}, {"ne": 0}, {"elems": None}, {"nnz": None}):
        rc, plan = make(**kw)
        assert rc == -1 and plan.value is None, kw
    for ident in (m.nverts, -1):  # found on the device before any use
        bad = e.clone()
        bad[3, 1] = ident
        rc, plan = make(elems=bad)
        assert rc == -1 and plan.value is None
    assert L.amg_p1_plan_device(2, m.nverts, len(m.elems), e.data_ptr(), C.byref(n), None, None) == -1
    rc, plan = make()
    assert rc == 0 and plan.value
    v = torch.zeros(max(n.value, 2 * m.nverts, m.nverts + 1, len(m.elems)), dtype=torch.float64, device="cuda")
    args = [plan, v.data_ptr(), e.data_ptr(), v.data_ptr(), v.data_ptr(), v.data_ptr(), v.data_ptr(), v.data_ptr()]
    for k in range(len(args)):
        assert L.amg_p1_assemble_planned(*[None if i == k else a for i, a in enumerate(args)]) == -1
    assert bool((v == 0).all())
    assert L.amg_p1_plan_destroy(plan) == 0
    assert L.amg_p1_plan_destroy(None) == 0
