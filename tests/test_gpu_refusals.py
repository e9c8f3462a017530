"""What a refused allocation or a refused input leaves: an error, no result that
looks like one, and a library that goes on working; and calls that were refused
for their size alone.  Allocations are refused by
the calling thread's allowance (stb_set_alloc_allowance, an internal function)."""
import contextlib
import ctypes

import numpy as np
import pytest

from paper_2103_16841_amd import inputs

pytestmark = pytest.mark.gpu

NO_MEMORY = 3


@pytest.fixture(scope="module")
def stb():
    import torch
    torch.cuda.init()
    from paper_2103_16841_amd import stb as s
    s.load()
    return s


@contextlib.contextmanager
def allowance(stb, nbytes):
    """Device allocations of this thread are refused beyond nbytes in all."""
    f = stb.load()._Z23stb_set_alloc_allowancel
    f.argtypes, f.restype = [ctypes.c_int64], None
    f(nbytes)
    try:
        yield
    finally:
        f(-1)


def test_refused_matrix_core_copy(stb):
    """Whichever allocation of the first 16-RHS product is refused, y is written
    or the call fails; the matrix has no copy then, and the next call works."""
    import torch
    ctx = stb.Context(0)
    mesh = inputs.icosphere_mesh(1, 8)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    W = torch.from_numpy(np.random.default_rng(0).standard_normal((mesh.nt, 16))).cuda()
    ref = stb.assemble_V(ctx, M).apply(W.cpu().numpy())
    A = stb.assemble_V(ctx, M)
    Y = torch.full_like(W, np.nan)
    torch.cuda.synchronize()
    refused, budget = 0, 0
    while True:
        ok = True
        with allowance(stb, budget):
            try:
                A.apply_dev(W.data_ptr(), Y.data_ptr(), 16)
            except stb.StbError as e:
                assert e.status == NO_MEMORY
                ok = False
        torch.cuda.synchronize()
        if ok:
            break
        refused += 1
        assert bool(torch.isnan(Y).all())
        # once the copy is there, only the product's own temporary is refused
        built = budget > 0 and stb.load().stb_apply16_noalloc(
            ctx.h, A.h, ctypes.c_void_p(W.data_ptr()), ctypes.c_void_p(Y.data_ptr()), None) == 0
        torch.cuda.synchronize()
        if built:
            assert np.array_equal(Y.cpu().numpy(), ref)
            Y.fill_(np.nan)
            torch.cuda.synchronize()
        budget = budget * 2 + 64
    assert refused >= 5
    assert np.array_equal(Y.cpu().numpy(), ref)
    A.close()
    M.close()
    ctx.close()


def test_one_candidate(stb):
    """A point and a panel by themselves, also where the point sees more pieces than
    a candidate has on average (close to a vertex: twelve and more)."""
    import oracle
    sphere = inputs.icosphere_mesh(0, 1, T=1.0)
    use = np.unique(sphere.tets[0])
    vtx = np.ascontiguousarray(sphere.vtx[use])
    tet = np.searchsorted(use, sphere.tets[:1]).astype(np.int32)
    normal = sphere.outward_normals()[:1]
    ctx = stb.Context(0)
    M = stb.Mesh(ctx, vtx, tet)
    M.set_normals(normal)
    rng = np.random.default_rng(0)
    pts = vtx[tet[0]][rng.integers(0, 4, 400)]
    step = 10.0 ** rng.uniform(-3, 0, (400, 1)) * rng.standard_normal((400, 4))
    step[:, 0] = np.abs(step[:, 0])
    pts = pts + step
    one, v = np.ones(1), rng.standard_normal(4)
    uS = np.concatenate([stb.potential_S(ctx, M, one, p[None]) for p in pts])
    uD = np.concatenate([stb.potential_D(ctx, M, v, p[None]) for p in pts])
    # the same points in one call: the same arithmetic per pair
    assert np.array_equal(uS, stb.potential_S(ctx, M, one, pts))
    assert np.array_equal(uD, stb.potential_D(ctx, M, v, pts))
    rS = oracle.potential(vtx, tet, one, pts)
    rD = oracle.potential_dl(vtx, tet, normal, v, pts)
    assert np.all(np.abs(uS - rS) <= 1e-10 * np.maximum(np.abs(rS), 1e-3 * np.abs(rS).max()))
    assert np.all(np.abs(uD - rD) <= 1e-10 * np.maximum(np.abs(rD), 1e-5 * np.abs(rD).max()))
    M.close()
    ctx.close()


@pytest.mark.parametrize("layer", ["S", "D"])
def test_potential_in_little_memory(stb, layer):
    """With ever more memory a potential is refused up to some point and computed
    from there on: the lists, and the double layer's sums beside them, take what
    there is, and the values do not depend on it."""
    mesh = inputs.icosphere_mesh(1, 8)
    pts = inputs.shell_points(300, mesh.T, seed=3)
    rng = np.random.default_rng(1)
    w = rng.standard_normal(mesh.nv if layer == "D" else mesh.nt)
    call = stb.potential_D if layer == "D" else stb.potential_S

    def run(nbytes):
        ctx = stb.Context(0)
        M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
        M.set_normals(mesh.outward_normals())
        try:
            with allowance(stb, nbytes):
                return call(ctx, M, w, pts)
        except stb.StbError as e:
            assert e.status == NO_MEMORY
            return None
        finally:
            M.close()
            ctx.close()
    ref = run(-1)
    refused, served = 0, 0
    budget = 1 << 16
    while served < 50:
        u = run(int(budget))
        if u is None:
            refused += 1
            assert served == 0, "%d bytes refused where less was enough" % budget
        else:
            served += 1
            assert np.array_equal(u, ref)
        budget *= 1.07
    assert refused > 10


def test_server_counts_the_cull(stb):
    """A potential's footprint has the cull's counts per point and panel segment in
    it: 100 points that no panel reaches (no candidates, no lists) on 2,880 panels,
    45 segments of 64."""
    mesh = inputs.icosphere_mesh(1, 12)
    ctx = stb.Context(0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    pts = inputs.shell_points(100, mesh.T, seed=1)
    pts[:, 0] = -1.0
    io = mesh.nt * 8 + 100 * (32 + 8 + 64 + 8)
    counts = 8 * 100 * 45
    for budget, fits in ((io + counts, False), (io + 2 * counts, False), (io + 2 * counts + 4096, True)):
        S = stb.Server(ctx, hbm_budget=budget, nslots=1)
        ticket = S.submit_potential(S.add_mesh(M), np.ones(mesh.nt), pts)
        if fits:
            assert np.array_equal(S.wait(ticket)[0], np.zeros(100))
        else:
            with pytest.raises(stb.StbError) as e:
                S.wait(ticket)
            assert e.value.status == NO_MEMORY
        S.close()
    M.close()
    ctx.close()


def test_store_without_a_product_plan(stb):
    """A large store whose product plan (where its rows cross the column parts) is
    refused keeps the product without one: the same sums in another order."""
    mesh = inputs.icosphere_mesh(2, 32)
    ctx = stb.Context(0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=1, n_g=2))
    plan = stb.load()._Z13stb_spmv_planP7stb_ctxP7stb_matP12ihipStream_t
    plan.argtypes = [ctypes.c_void_p] * 3
    w = np.random.default_rng(2).standard_normal(A.n)
    y = A.apply(w)
    with allowance(stb, 0):
        assert plan(ctx.h, A.h, None) == 0
    z = A.apply(w)
    rowptr, cols, vals = A.export()
    from scipy.sparse import csr_matrix
    scale = csr_matrix((np.abs(vals), cols, rowptr), shape=(A.n, A.n)) @ np.abs(w)
    terms = np.diff(rowptr)
    assert not np.array_equal(y, z)
    # either order: at most (terms) eps of the terms' size
    assert np.all(np.abs(y - z) <= 2 * terms * 2.0 ** -53 * scale)
    assert plan(ctx.h, A.h, None) == 0
    assert np.array_equal(A.apply(w), y)
    A.close()
    M.close()
    ctx.close()
