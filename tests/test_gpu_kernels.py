"""Small tests of single kernels at the sizes where they can go wrong: edges of
tiles and parts, remainders, the smallest and largest of a dispatch's range.
References are plain numpy on the library's own exported values, or the oracle."""
import numpy as np
import pytest

from paper_2103_16841_amd import inputs

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -53


@pytest.fixture(scope="module")
def stb():
    import torch
    torch.cuda.init()
    from paper_2103_16841_amd import stb as s
    s.load()
    return s


@pytest.fixture(scope="module")
def ctx(stb):
    c = stb.Context(0)
    yield c
    c.close()


def _rows_of(A, rows):
    """Dense rows of a matrix through stb_mat_get."""
    cols = np.tile(np.arange(A.n, dtype=np.int32), len(rows))
    return A.get(np.repeat(np.asarray(rows, dtype=np.int32), A.n), cols).reshape(len(rows), A.n)


# one column part (15,360 panels), two (30,720) and three (40,320, the last part's
# rows mostly empty before the late slabs); 11,520 panels stay below the limit
@pytest.mark.parametrize("level,slabs", [(1, 48), (2, 16), (2, 32), (2, 42)])
def test_product_with_column_parts(stb, ctx, level, slabs):
    mesh = inputs.icosphere_mesh(level, slabs)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=1, n_g=2))
    rng = np.random.default_rng(0)
    # the first rows (nearly empty), the last, both sides of the workgroups' strides
    rows = np.unique(np.concatenate([[0, 1, 15, 16, 4095, 4096, A.n - 1], rng.integers(0, A.n, 9)]))
    D = _rows_of(A, rows)
    for nrhs in (1, 3):
        W = rng.standard_normal((A.n, nrhs) if nrhs > 1 else A.n)
        Y = A.apply(W)
        ref = D @ W
        # any order of summation: at most (terms) eps of the terms' size
        bound = (D != 0).sum(1) * EPS * 2
        scale = np.abs(D) @ np.abs(W)
        assert np.all(np.abs(Y[rows] - ref) <= (bound[:, None] * scale if nrhs > 1 else bound * scale))
    A.close()
    M.close()


# fewer unknowns than a chunk of the dot products, a remainder chunk, restarts
# shorter and longer than the vectors subtracted at once
@pytest.mark.parametrize("slabs,restart", [(1, 1), (6, 5), (6, 100), (18, 8), (18, 9), (18, 100)])
def test_gmres_restarts(stb, ctx, slabs, restart):
    mesh = inputs.icosphere_mesh(0, slabs, T=2.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M)
    D = A.to_dense()
    b = D @ np.random.default_rng(slabs).standard_normal(A.n)
    x, its, rel = stb.solve_gmres(ctx, A, b, restart=restart, maxit=40, rtol=1e-10)
    assert its <= 40
    # the reported residual is the true one: the product's rounding error aside
    true = np.linalg.norm(b - D @ x) / np.linalg.norm(b)
    slack = A.n * EPS * 2 * np.linalg.norm(np.abs(D) @ np.abs(x)) / np.linalg.norm(b)
    assert abs(true - rel) <= slack + 1e-12 * rel
    # no more work than asked: one more product than steps at most, and a longer
    # search never ends with a larger residual
    x2, its2, rel2 = stb.solve_gmres(ctx, A, b, restart=restart, maxit=39, rtol=1e-10)
    assert its2 <= 39 and rel <= rel2 * (1 + 1e-9) + slack
    if restart == 100 and slabs <= 6:
        # the minimal residual over the Krylov space itself
        k = min(its, 20)
        x3, its3, rel3 = stb.solve_gmres(ctx, A, b, restart=restart, maxit=k, rtol=1e-14)
        Q = np.zeros((A.n, k))
        v = b / np.linalg.norm(b)
        for i in range(k):
            Q[:, i] = v
            v = D @ v
            for _ in range(2):
                v -= Q[:, :i + 1] @ (Q[:, :i + 1].T @ v)
            v /= np.linalg.norm(v)
        z, *_ = np.linalg.lstsq(D @ Q, b, rcond=None)
        best = np.linalg.norm(b - D @ (Q @ z)) / np.linalg.norm(b)
        assert abs(rel3 - best) <= 1e-8 * best + slack


# K = 60 (fewer rows than a panel step's workgroup, a last panel of 12 columns), 12 and
# 960 by the slabs' triangles; 1,280 and 5,120 take two and eight rows per lane
@pytest.mark.parametrize("level,slabs", [(-1, 3), (0, 5), (2, 3), (3, 2)])
def test_marching_equals_dense_solve(stb, ctx, level, slabs):
    if level < 0:
        mesh = inputs.cube_mesh(S=slabs, T=1.0)
    else:
        pts, tris = inputs.icosphere(level)
        mesh = inputs.extrude(pts, tris, slabs, 0.5 * slabs)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=2, n_g=8))
    rng = np.random.default_rng(level + 5)
    b = A.apply(rng.standard_normal(A.n))
    x, info = stb.solve_mot(ctx, M, A, b)
    K = A.n // slabs
    assert info["slabs"] == slabs and info["panels_per_slab"] == K
    # the same marching in numpy: slab 0's diagonal block on every slab
    lo = mesh.tet_coords()[:, :, 0].min(1)
    idx = [np.where(np.isclose(lo, n * mesh.T / slabs))[0] for n in range(slabs)]
    block = lambda i, j: A.get(np.repeat(i, len(j)).astype(np.int32), np.tile(j, len(i)).astype(np.int32)).reshape(len(i), -1)
    D = block(idx[0], idx[0])
    ref = np.zeros(A.n)
    for n in range(slabs):
        r = b[idx[n]].copy()
        for m in range(n):
            r -= block(idx[n], idx[m]) @ ref[idx[m]]
        ref[idx[n]] = np.linalg.solve(D, r)
    # a solve by an explicit inverse: a few K eps cond(D) of the block's size
    cond = np.linalg.cond(D)
    assert np.linalg.norm(x - ref) <= 8 * K * EPS * cond ** 2 * np.linalg.norm(ref)


# odd and even node counts; points on both sides of the logarithm series' limit
# (far: gaps of a tenth of r, near: gaps of several r), and in panels' planes
@pytest.mark.parametrize("n_g", [2, 3, 16, 33])
def test_double_layer_nodes(stb, ctx, n_g):
    import oracle
    mesh = inputs.icosphere_mesh(1, 6, T=3.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    M.set_normals(mesh.outward_normals())
    v = np.random.default_rng(1).standard_normal(mesh.nv)
    cen = mesh.tet_coords().mean(axis=1)[::37]
    near = cen + np.concatenate([np.full((len(cen), 1), 0.3), 1e-3 * mesh.outward_normals()[::37]], axis=1)
    flat = cen + np.array([0.4, 0.0, 0.0, 0.0])
    pts = np.concatenate([inputs.shell_points(60, mesh.T, seed=2), near, flat])
    u = stb.potential_D(ctx, M, v, pts, params=stb.default_params(n_g=n_g))
    ref = oracle.potential_dl(mesh.vtx, mesh.tets, mesh.outward_normals(), v, pts, n_g=n_g)
    # the double layer's parity bound: 1e-10 relative above 1e-5 of the largest value
    assert np.all(np.abs(u - ref) <= 1e-10 * np.maximum(np.abs(ref), 1e-5 * np.abs(ref).max()))


# odd and even node counts; all lit pairs (also near ones, with pieces longer than
# pi) and far ones only; panels with faces of constant time, tied with the range's ends
@pytest.mark.parametrize("n_g", [2, 3, 33])
@pytest.mark.parametrize("eta", [0.0, 2.0])
def test_mixed_recipe_nodes(stb, ctx, n_g, eta):
    mesh = inputs.icosphere_mesh(1, 4, T=3.0, jitter=0.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    par = lambda e: stb.default_params(m_q=2, n_g=n_g, prec=stb.STB_MIXED, eta_far=e)
    A = stb.assemble_V(ctx, M, par(eta))
    assert ctx.kernel_times()["nodes_fp32"][2] > 0
    B = stb.assemble_V(ctx, M, par(1e300))   # no far pairs: FP64 through the same points
    (ra, ca, va), (rb, cb, vb) = A.export(), B.export()
    assert np.array_equal(ra, rb) and np.array_equal(ca, cb)
    # the mixed assembly's bound per entry
    assert np.all(np.abs(va - vb) <= 1e-6 * np.abs(vb))


# blocks of fewer rows than 16, chains shorter than a group of loads, remainders
# of groups, and long chains; the quads' stored values against the CSR's
@pytest.mark.parametrize("level,slabs", [(0, 1), (0, 3), (1, 5), (2, 9)])
def test_sixteen_right_hand_sides(stb, ctx, level, slabs):
    mesh = inputs.icosphere_mesh(level, slabs)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=1, n_g=2))
    rows = np.unique(np.concatenate([np.arange(min(A.n, 40)), np.arange(max(A.n - 40, 0), A.n)]))
    D = _rows_of(A, rows)
    W = np.random.default_rng(3).standard_normal((A.n, 16))
    Y = A.apply(W)
    ref = D @ W
    # products of rounded factors (2 units each) summed in FP32: terms + 3 units of the terms' size
    bound = ((D != 0).sum(1) + 3)[:, None] * 2.0 ** -24
    assert np.all(np.abs(Y[rows] - ref) <= bound * (np.abs(D) @ np.abs(W)))
    # every column alone: unit vectors pick single entries, exactly the FP32 values
    E = np.zeros((A.n, 16))
    pick = np.linspace(0, A.n - 1, 16).astype(int)
    E[pick, np.arange(16)] = 1.0
    assert np.array_equal(A.apply(E)[rows], D[:, pick].astype(np.float32).astype(np.float64))


# one row, both sides of a wavefront's 16 and a workgroup's 64 rows, panels that
# are no multiple of 64, points on light cones of vertices (the bounds' ends), and
# a mesh far from the origin, where single precision decides little
@pytest.mark.parametrize("npts", [1, 15, 17, 63, 65, 130])
@pytest.mark.parametrize("shift", [0.0, 64.0])
def test_cull_rows_and_segments(stb, ctx, npts, shift):
    import oracle
    mesh = inputs.icosphere_mesh(0, 3, T=2.0)
    vtx = np.ascontiguousarray(mesh.vtx + shift)
    M = stb.Mesh(ctx, vtx, mesh.tets)
    w = np.random.default_rng(2).standard_normal(mesh.nt)
    pts = inputs.shell_points(npts, mesh.T, seed=npts)
    k = np.arange(0, npts, 3)   # t - t_v = |x - x_v| for a vertex v
    v = mesh.vtx[k % mesh.nv]
    pts[k, 0] = v[:, 0] + np.linalg.norm(pts[k, 1:] - v[:, 1:], axis=1)
    pts = pts + shift
    u = stb.potential_S(ctx, M, w, pts)
    ref, mag = oracle.potential(vtx, mesh.tets, w, pts), oracle.potential(vtx, mesh.tets, np.abs(w), pts)
    # the potential's parity bound, at coordinates known to 64 eps when shifted
    assert np.all(np.abs(u - ref) <= 1e-10 * np.maximum(mag, 1e-3 * mag.max()))


# fewer nodes than a piece's lanes, one more, and two rounds of them; points whose
# cones meet a panel's plane in whole circles (no breakpoints) and in short pieces
@pytest.mark.parametrize("n_g", [2, 15, 17, 33])
def test_full_evaluation_nodes(stb, ctx, n_g):
    import oracle
    mesh = inputs.icosphere_mesh(0, 4, T=4.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    w = np.random.default_rng(4).standard_normal(mesh.nt)
    cen = mesh.tet_coords().mean(axis=1)
    pts = np.concatenate([cen + [1e-2, 0, 0, 0], cen + [0.2, 1e-3, 0, 0], inputs.shell_points(40, mesh.T, seed=9)])
    u = stb.potential_S(ctx, M, w, pts, stb.default_params(n_g=n_g))
    assert ctx.path_counts()["full"] > 0
    ref = oracle.potential(mesh.vtx, mesh.tets, w, pts, n_g=n_g)
    mag = oracle.potential(mesh.vtx, mesh.tets, np.abs(w), pts, n_g=n_g)
    # the potential's parity bound
    assert np.all(np.abs(u - ref) <= 1e-10 * np.maximum(mag, 1e-3 * mag.max()))


# rows shorter than a wavefront (every wavefront spans rows), about one, several;
# faces whose candidates start before, with and after the row's
@pytest.mark.parametrize("level,slabs", [(0, 1), (0, 3), (1, 2), (1, 5)])
def test_entries_from_face_sums(stb, ctx, level, slabs):
    from _tol import assert_entries, oracle_rows
    mesh = inputs.icosphere_mesh(level, slabs, T=2.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M)
    rows = np.unique(np.linspace(0, A.n - 1, 12).astype(int))
    ref, mag, pert = oracle_rows(mesh.vtx, mesh.tets, rows=rows)
    assert_entries(_rows_of(A, rows), ref, mag, pert)


# the matrix-core copy entry by entry: one row, a last block of one row and of 15, a
# last quad of one column, one pass of the fill and several, empty rows
@pytest.mark.parametrize("level,ntri,slabs", [(0, 1, 1), (0, 5, 1), (0, 17, 1), (0, 19, 3), (1, 67, 3), (1, 80, 8)])
def test_every_entry_of_the_matrix_core_copy(stb, ctx, level, ntri, slabs):
    pts, tris = inputs.icosphere(level)
    use = np.unique(tris[:ntri])
    mesh = inputs.extrude(pts[use], np.searchsorted(use, tris[:ntri]).astype(tris.dtype), slabs, 4.0)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=1, n_g=4))
    D = A.to_dense().astype(np.float32).astype(np.float64)
    for c in range(0, A.n, 16):
        E = np.zeros((A.n, 16))
        k = np.arange(c, min(c + 16, A.n))
        E[k, k - c] = 1.0
        assert np.array_equal(A.apply(E)[:, :len(k)], D[:, k]), c
    A.close()
    M.close()


# the stores of test_product_with_column_parts are on the sides of the limit that it
# means: 2^24 entries; parts of at most 19,200 columns.  A large store's sums run by
# parts, so the order of its rows' sums is the store's own: each part's entries as
# they are summed in a row of 64 lanes, then the parts
@pytest.mark.parametrize("level,slabs,parts", [(1, 48, 0), (2, 16, 1), (2, 32, 2), (2, 42, 3)])
def test_column_part_stores_pass_the_limit(stb, ctx, level, slabs, parts):
    mesh = inputs.icosphere_mesh(level, slabs)
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    A = stb.assemble_V(ctx, M, stb.default_params(m_q=1, n_g=2))
    assert (A.n_stored >= 2 ** 24) == (parts > 0)
    w = np.random.default_rng(1).standard_normal(A.n)
    y = A.apply(w)
    if parts:
        width = -(-A.n // parts)
        assert -(-A.n // 19200) == parts
        row = A.n - 1
        v = A.get(np.full(A.n, row, dtype=np.int32), np.arange(A.n, dtype=np.int32))
        c = np.nonzero(v)[0]
        y_parts = A.apply(np.where(np.arange(A.n) < width, w, 0.0))[row]
        for p in range(1, parts):
            y_parts += A.apply(np.where(np.arange(A.n) // width == p, w, 0.0))[row]
        # a part alone gives that part's sum and exact zeros elsewhere
        assert y[row] == y_parts and len(c) > 64
    A.close()
    M.close()


# few candidates (their combos listed in one launch), both sides of its 4,096, and
# chunks of few candidates by short lists, which overflow: a point's value is the
# same in every call
@pytest.mark.parametrize("layer", ["S", "D"])
def test_potentials_do_not_depend_on_the_call(stb, layer):
    mesh = inputs.icosphere_mesh(1, 13)
    rng = np.random.default_rng(7)
    pts = inputs.shell_points(60, mesh.T, seed=8)
    w = rng.standard_normal(mesh.nv if layer == "D" else mesh.nt)
    call = stb.potential_D if layer == "D" else stb.potential_S
    c = stb.Context(0)
    M = stb.Mesh(c, mesh.vtx, mesh.tets)
    M.set_normals(mesh.outward_normals())
    ref = call(c, M, w, pts)
    assert c.lit_search()["candidates"] > 4096 > 0
    sizes = set()
    for k in (1, 2, 5, 9, 20):
        u = np.concatenate([call(c, M, w, pts[i:i + k]) for i in range(0, 60, k)])
        sizes.add(c.lit_search()["candidates"] > 4096)
        assert np.array_equal(u, ref), k
    for limits in ((64, 64, 64), (5000, 0, 0), (0, 100, 0), (0, 0, 300)):
        stb.set_pair_lists(c, *limits)
        assert np.array_equal(call(c, M, w, pts), ref), limits
    assert sizes == {False, True}
    M.close()
    c.close()
