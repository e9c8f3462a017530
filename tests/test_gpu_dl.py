"""The double-layer potential (eq. dlp) and the energetic forms b_I, b_K
(eq. int_bform) on the GPU, through the C ABI, against the FP64 oracle
(same phi-rule; tolerances as for the single layer: relative 1e-10 above
1e-5 of the largest value), and against what the mathematics fixes:
Gauss's law on closed surfaces, K 1 = -1/2 on them, Kirchhoff's
representation of a wave from an outside point source, and the direct
method (eq. df_dir) converging for the paper's exterior example.
"""
import numpy as np
import pytest

import oracle
from paper_2103_16841_amd import inputs
from _pins import (point_source_wave, point_source_wave_dn, BIG_TET, BIG_TET_POINTS,
                   big_tet_closed_form)

pytestmark = pytest.mark.gpu

RTOL = 1e-10
FLOOR = 1e-5


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


def _mesh(stb, ctx, mesh):
    m = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    m.set_normals(mesh.outward_normals())
    return m


def _check(a, ref, what):
    scale = np.abs(ref).max()
    err = np.abs(a - ref) / np.maximum(np.abs(ref), FLOOR * scale)
    k = int(np.argmax(err))
    print("%s: %d values, max |ref| %.3e, worst rel err %.3e (gpu %.17g oracle %.17g)"
          % (what, ref.size, scale, err.flat[k], a.flat[k], ref.flat[k]), flush=True)
    assert err.max() <= RTOL


def test_hat_values_vs_oracle(stb, ctx):
    mesh = inputs.icosphere_mesh(level=1, S=4, T=3.0, jitter=0.2, seed=7)
    m = _mesh(stb, ctx, mesh)
    nrm = mesh.outward_normals()
    rng = np.random.default_rng(11)
    opts, _, _ = stb.outer_points(ctx, m)
    # outer points of random panels (on the surface), near-surface and shell points
    k = 400
    src = rng.integers(0, mesh.nt, k)
    on = opts[src, rng.integers(0, 18, k)]
    d = rng.standard_normal((k, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    near = np.concatenate([rng.uniform(0.5, 3.0, (k, 1)), d * rng.uniform(0.9, 1.1, (k, 1))], axis=1)
    shell = inputs.shell_points(k, mesh.T, rmin=1.2, rmax=2.0, seed=12)
    pts = np.concatenate([on, near, shell])
    # pair every point with panels its light cone reaches (and some it does not)
    pan = rng.integers(0, mesh.nt, pts.shape[0])
    got = stb.inner_values_D(ctx, m, pts, pan)
    ref = np.zeros_like(got)
    eye = np.eye(4)
    for i in range(pts.shape[0]):
        T = mesh.vtx[mesh.tets[pan[i]]]
        for q in range(4):
            ref[i, q] = oracle.inner_dl(pts[i], T, nrm[pan[i]], eye[q])
    assert np.count_nonzero(ref) > 400
    assert np.all((got == 0.0) == (ref == 0.0))
    _check(got, ref, "hat values")


def test_potential_vs_oracle(stb, ctx):
    mesh = inputs.icosphere_mesh(level=1, S=8, T=4.0, jitter=0.2, seed=5)
    m = _mesh(stb, ctx, mesh)
    v = inputs.density_normal(mesh.nv, seed=3)
    rng = np.random.default_rng(8)
    d = rng.standard_normal((100, 3))
    d /= np.linalg.norm(d, axis=1, keepdims=True)
    near = np.concatenate([rng.uniform(0.5, 4.0, (100, 1)), d * rng.uniform(0.3, 1.2, (100, 1))], axis=1)
    pts = np.concatenate([inputs.shell_points(200, mesh.T, seed=4), near])
    u = stb.potential_D(ctx, m, v, pts)
    uo = oracle.potential_dl(mesh.vtx, mesh.tets, mesh.outward_normals(), v, pts)
    _check(u, uo, "potential")


def test_gauss_closed_surface(stb, ctx):
    mesh = inputs.icosphere_mesh(level=2, S=4, T=6.0, jitter=0.2, seed=4)
    m = _mesh(stb, ctx, mesh)
    ones = np.ones(mesh.nv)
    inside = np.array([[5.0, 0.0, 0.0, 0.0], [5.0, 0.3, -0.2, 0.4], [4.8, -0.5, 0.1, 0.2]])
    outside = np.array([[5.0, 1.6, 0.0, 0.3], [5.5, -0.9, 1.3, -0.8]])
    for n_g, tol in ((64, 1e-10), (16, 2e-7)):
        p = stb.default_params(n_g=n_g)
        u_in = stb.potential_D(ctx, m, ones, inside, params=p)
        u_out = stb.potential_D(ctx, m, ones, outside, params=p)
        print("n_g %d: D1 inside + 1 = %s, outside = %s" % (n_g, u_in + 1.0, u_out), flush=True)
        assert np.all(np.abs(u_in + 1.0) <= tol)
        assert np.all(np.abs(u_out) <= tol)


def test_kirchhoff_representation(stb, ctx):
    """Inside the sphere u = S(du/dn) - D(u) (Kirchhoff's formula for the
    interior with the outward normal): D of the vertex interpolant of u
    (V_h^1) and S of du/dn at the panel centroids (S_h^0)."""
    pts = np.array([[3.5, 0.0, 0.0, 0.3], [3.2, 0.2, -0.3, 0.0], [3.8, -0.2, 0.1, -0.4]])
    exact = point_source_wave(pts)
    errs = []
    for level, S in ((2, 16), (3, 32)):
        mesh = inputs.icosphere_mesh(level=level, S=S, T=4.0, jitter=0.0, seed=0)
        m = _mesh(stb, ctx, mesh)
        nrm = mesh.outward_normals()
        cen = mesh.vtx[mesh.tets].mean(axis=1)
        rep = (stb.potential_S(ctx, m, point_source_wave_dn(cen, nrm), pts)
               - stb.potential_D(ctx, m, point_source_wave(mesh.vtx), pts))
        err = np.abs(rep - exact).max() / np.abs(exact).max()
        print("case: sphere level %d S %d N %d: representation error %.3e" % (level, S, mesh.nt, err),
              flush=True)
        errs.append(err)
    assert errs[1] < 0.01 and errs[1] < 0.3 * errs[0]


def test_bench_workload_sampled(stb, ctx):
    """The bench's double-layer leg (icosphere level 2, 32 slabs, 1,000 shell
    points in one launch) against the oracle on a sample of the points."""
    mesh = inputs.icosphere_mesh()
    m = _mesh(stb, ctx, mesh)
    v = inputs.density_normal(mesh.nv, seed=9)
    pts = inputs.shell_points(1000, mesh.T, seed=1)
    u = stb.potential_D(ctx, m, v, pts)
    idx = np.arange(0, 1000, 125)
    uo = oracle.potential_dl(mesh.vtx, mesh.tets, mesh.outward_normals(), v, pts[idx])
    _check(u[idx], uo, "bench workload sample")


def test_energetic_forms_vs_oracle(stb, ctx):
    """c_id b_I(v, phi_i) + b_K(v, phi_i) (outer rule of eq. int_bform) on
    sampled rows against the oracle, random V_h^1 density."""
    mesh = inputs.icosphere_mesh(level=1, S=4, T=3.0, jitter=0.2, seed=7)
    m = _mesh(stb, ctx, mesh)
    v = inputs.density_normal(mesh.nv, seed=13)
    got = stb.dl_energetic(ctx, m, v, c_id=0.5)
    rows = np.arange(3, mesh.nt, 41)
    ref = oracle.dl_energetic_rows(mesh.vtx, mesh.tets, mesh.outward_normals(), v, rows, c_id=0.5)
    _check(got[rows], ref, "energetic forms, sampled rows")


def test_energetic_forms_exact(stb, ctx):
    """On a closed polyhedron K 1 = -1/2 inside its faces, so in the static
    regime b_K(tau, phi_i) = -1/2 sum_q w_iq t_q; b_I of an affine function
    is its outer-rule sum."""
    mesh = inputs.icosphere_mesh(level=1, S=3, T=6.0, jitter=0.2, seed=4)
    m = _mesh(stb, ctx, mesh)
    ct = mesh.centroid_times()
    rows = np.where((ct > 3.0) & (ct < mesh.T - 0.5))[0]
    pts, w, n = stb.outer_points(ctx, m)
    bk = stb.dl_energetic(ctx, m, mesh.vtx[:, 0].copy(), c_id=0.0, params=stb.default_params(n_g=64))
    ex = -0.5 * np.einsum("iq,iq->i", w, pts[:, :, 0])
    print("b_K(tau) worst abs err %.3e over %d static rows" % (np.abs(bk - ex)[rows].max(), rows.size),
          flush=True)
    assert np.all(np.abs(bk - ex)[rows] <= 1e-12)
    a = np.array([0.3, -0.7, 0.4, 1.1])
    va = 0.2 + mesh.vtx @ a
    bi = stb.dl_energetic(ctx, m, va, c_id=1.0) - stb.dl_energetic(ctx, m, va, c_id=0.0)
    exi = np.einsum("iq,iq->i", w, 0.2 + pts @ a)
    assert np.all(np.abs(bi - exi) <= 1e-14)


def test_projection_vs_oracle(stb, ctx):
    """Q_h^1: the rule's points and weights, and the projection of a smooth
    function, against the oracle; a V_h^1 function is reproduced."""
    mesh = inputs.icosphere_mesh(level=1, S=4, T=3.0, jitter=0.2, seed=7)
    m = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    P, W = stb.l2_points(ctx, m)
    Po = np.array([oracle.l2_points(mesh.vtx[mesh.tets[j]])[0] for j in range(mesh.nt)])
    Wo = np.array([oracle.l2_points(mesh.vtx[mesh.tets[j]])[1] for j in range(mesh.nt)])
    assert np.abs(P - Po).max() <= 1e-14 and np.abs(W - Wo).max() <= 1e-15
    f = lambda p: np.sin(p[..., 0]) * np.cos(2.0 * p[..., 1]) + p[..., 2] * p[..., 3]
    c, its = stb.project_V1(ctx, m, f(P), mesh.nv)
    co = oracle.l2_projection(mesh.vtx, mesh.tets, f(Po))
    print("projection: %d CG steps, worst abs err %.3e (max |c| %.3f)" % (its, np.abs(c - co).max(),
                                                                          np.abs(co).max()), flush=True)
    assert np.abs(c - co).max() <= 1e-10 * np.abs(co).max()
    a = np.array([0.3, -0.7, 0.4, 1.1])
    c1, _ = stb.project_V1(ctx, m, 0.2 + P @ a, mesh.nv)
    assert np.abs(c1 - (0.2 + mesh.vtx @ a)).max() <= 1e-12


def test_direct_method_exterior(stb, ctx):
    """The direct method (eq. df_dir) for the exterior problem of the paper's
    last example: a spherical wave mu(t - |x - y_S|) / |x - y_S| from y_S
    inside, mu(t) = t^3 e^-t; Dirichlet data projected, Q_h^1 g, the
    right-hand side -1/2 b_I(Q g) + b_K(Q g), GMRES for the Neumann trace,
    then u_h = D Q g - S w_h outside.  Both errors fall under refinement."""
    ys = np.array([-0.1, -0.2, -0.3])

    def mu(t):
        tp = np.maximum(t, 0.0)
        return np.where(t > 0.0, tp ** 3 * np.exp(-tp), 0.0)

    def mu_dt(t):
        tp = np.maximum(t, 0.0)
        return np.where(t > 0.0, (3.0 * tp ** 2 - tp ** 3) * np.exp(-tp), 0.0)

    def u(p):
        r = np.linalg.norm(p[..., 1:] - ys, axis=-1)
        return mu(p[..., 0] - r) / r

    def u_dn(p, nrm):
        y = p[..., 1:]
        r = np.linalg.norm(y - ys, axis=-1)
        tr = p[..., 0] - r
        g = (-mu_dt(tr) / r - mu(tr) / (r * r))[..., None] * (y - ys) / r[..., None]
        return np.einsum("...i,...i->...", g, nrm)

    far = np.array([[4.0, 1.5, 0.0, 0.3], [4.0, 0.2, -1.6, 0.0], [4.0, -1.2, 0.9, -0.6]])
    errs, ferrs = [], []
    for level, S in ((1, 8), (2, 16)):
        mesh = inputs.icosphere_mesh(level=level, S=S, T=4.0, jitter=0.0, seed=0)
        m = _mesh(stb, ctx, mesh)
        nrm = mesh.outward_normals()
        A = stb.assemble_V(ctx, m)
        P, _ = stb.l2_points(ctx, m)
        g, _ = stb.project_V1(ctx, m, u(P), mesh.nv)
        b = stb.dl_energetic(ctx, m, g, c_id=-0.5)
        x, its, rr = stb.solve_gmres(ctx, A, b, restart=100, maxit=20000, rtol=1e-10)
        cen = mesh.vtx[mesh.tets].mean(axis=1)
        ex = u_dn(cen, nrm)
        errs.append(np.linalg.norm(x - ex) / np.linalg.norm(ex))
        uh = stb.potential_D(ctx, m, g, far) - stb.potential_S(ctx, m, x, far)
        ferrs.append(np.max(np.abs(uh - u(far)) / np.abs(u(far))))
        print("case: sphere level %d S %d N %d: GMRES %d products, Neumann rel L2 error %.3e, "
              "field rel error %.3e" % (level, S, mesh.nt, its, errs[-1], ferrs[-1]), flush=True)
        A.close()
    assert errs[1] < 0.6 * errs[0] and errs[1] < 0.08
    assert ferrs[1] < 0.5 * ferrs[0] and ferrs[1] < 0.03


def test_device_pointer_path(stb, ctx):
    """stb_potential_D_dev with device-resident vertex values, points and
    output equals the host entry point bit for bit."""
    import torch
    mesh = inputs.icosphere_mesh(level=1, S=4, T=3.0, jitter=0.2, seed=7)
    m = _mesh(stb, ctx, mesh)
    v = inputs.density_normal(mesh.nv, seed=21)
    pts = inputs.shell_points(200, mesh.T, rmin=1.1, rmax=2.5, seed=22)
    dev = torch.device("cuda:0")
    vd = torch.from_numpy(v).to(dev)
    pd = torch.from_numpy(pts).to(dev)
    ud = torch.empty(pts.shape[0], dtype=torch.float64, device=dev)
    torch.cuda.synchronize()
    stb.potential_D_dev(ctx, m, vd.data_ptr(), pts.shape[0], pd.data_ptr(), ud.data_ptr())
    torch.cuda.synchronize()
    u = stb.potential_D(ctx, m, v, pts)
    assert np.array_equal(ud.cpu().numpy(), u)
    assert np.count_nonzero(u) > 100


def test_projection_arguments(stb, ctx):
    mesh = inputs.icosphere_mesh(level=0, S=2, T=2.0, jitter=0.0, seed=0)
    m = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    P, W = stb.l2_points(ctx, m)
    assert P.shape == (mesh.nt, 27, 4) and abs(W.sum() - _area_times_T(mesh)) <= 1e-12 * W.sum()
    with pytest.raises(ValueError):
        stb.project_V1(ctx, m, np.ones(mesh.nt * 27 - 1), mesh.nv)
    g = np.ones(mesh.nt * 27)
    g[5] = np.nan
    with pytest.raises(stb.StbError):
        stb.project_V1(ctx, m, g, mesh.nv)
    c, its = stb.project_V1(ctx, m, np.zeros(mesh.nt * 27), mesh.nv)
    assert its == 0 and np.all(c == 0.0)


def _area_times_T(mesh):
    """|Sigma| = T x the area of the spatial triangles (extruded meshes)."""
    X = mesh.vtx[:, 1:]
    tri = X[np.asarray(mesh.tri)]
    area = 0.5 * np.linalg.norm(np.cross(tri[:, 1] - tri[:, 0], tri[:, 2] - tri[:, 0]), axis=1).sum()
    return area * mesh.T


def test_periodic_case_one_panel(stb, ctx):
    """A one-panel mesh whose cone sections have no breakpoints (the
    periodic rule of both stages) against the closed form."""
    m = stb.Mesh(ctx, BIG_TET, np.array([[0, 1, 2, 3]]))
    vv = np.array([1.0, 2.0, 3.0, 4.0])
    for sgn in (1.0, -1.0):
        m.set_normals(np.array([[0.0, 0.0, sgn]]))
        u = stb.potential_D(ctx, m, vv, np.array(BIG_TET_POINTS))
        ref = np.array([big_tet_closed_form(x, vv, sgn) for x in BIG_TET_POINTS])
        assert np.all(np.abs(u - ref) <= 1e-13)
        h = stb.inner_values_D(ctx, m, np.array(BIG_TET_POINTS), np.zeros(3, dtype=np.int32))
        assert np.all(np.abs(h @ vv - ref) <= 1e-13)


def test_points_on_vertex_light_cones(stb, ctx):
    """Points exactly on the light cones of mesh vertices (the cone passes
    through a panel vertex: a breakpoint that only the closed-edge events
    give), single and double layer against the oracle."""
    mesh = inputs.icosphere_mesh(level=1, S=8, T=4.0, jitter=0.0, seed=0)
    m = _mesh(stb, ctx, mesh)
    rng = np.random.default_rng(31)
    pts = []
    for _ in range(60):
        v = mesh.vtx[rng.integers(0, mesh.nv)]
        d = rng.standard_normal(3)
        d /= np.linalg.norm(d)
        r = rng.choice([0.5, 1.0, 1.5, 2.0])
        pts.append([v[0] + r, *(v[1:] + r * d)])
    pts.append([4.0, 0.2, -1.6, 0.0])
    pts = np.array(pts)
    w = inputs.density_normal(mesh.nt, seed=32)
    v = inputs.density_normal(mesh.nv, seed=33)
    _check(stb.potential_S(ctx, m, w, pts), oracle.potential(mesh.vtx, mesh.tets, w, pts), "single layer")
    _check(stb.potential_D(ctx, m, v, pts),
           oracle.potential_dl(mesh.vtx, mesh.tets, mesh.outward_normals(), v, pts), "double layer")


def test_arguments(stb, ctx):
    mesh = inputs.icosphere_mesh(level=0, S=2, T=2.0, jitter=0.0, seed=0)
    m = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    pts = np.array([[1.5, 0.0, 0.0, 0.0]])
    with pytest.raises(stb.StbError):
        stb.potential_D(ctx, m, np.ones(mesh.nv), pts)        # no normals yet
    nrm = mesh.outward_normals()
    bad = nrm.copy()
    bad[5] = np.cross(bad[5], [0.3, 0.1, 0.9])               # in the panel's plane
    with pytest.raises(stb.StbError):
        m.set_normals(bad)
    with pytest.raises(ValueError):
        m.set_normals(nrm[:-1])
    m.set_normals(nrm)
    assert stb.potential_D(ctx, m, np.ones(mesh.nv), np.zeros((0, 4))).shape == (0,)
    u1 = stb.potential_D(ctx, m, np.ones(mesh.nv), pts)
    m.set_normals(-nrm)
    u2 = stb.potential_D(ctx, m, np.ones(mesh.nv), pts)
    assert u1[0] == -u2[0] and u1[0] < -0.9


# A root takes about a dozen roundings here and a dozen in the oracle, and the
# nodes' errors partly cancel: most values of single pairs agree within 24 eps.
# (Reciprocals and square roots one Newton step short, 10 and 19 eps a time and
# always to the same side, do not.)
@pytest.mark.parametrize("panel", [0, 1, 2, 30])
@pytest.mark.parametrize("n_g", [2, 16])
def test_pairs_to_rounding(stb, ctx, panel, n_g):
    sphere = inputs.icosphere_mesh(0, 2, T=2.0)
    use = np.unique(sphere.tets[panel])
    vtx = np.ascontiguousarray(sphere.vtx[use])
    tet = np.searchsorted(use, sphere.tets[panel:panel + 1]).astype(np.int32)
    normal = sphere.outward_normals()[panel:panel + 1]
    M = stb.Mesh(ctx, vtx, tet)
    M.set_normals(normal)
    # points whose cones pass through the panel near its centre
    pts = inputs.shell_points(4000, 1.0, seed=5)
    c = vtx.mean(0)
    pts[:, 0] = c[0] + np.linalg.norm(pts[:, 1:] - c[1:], axis=1) + np.random.default_rng(3).uniform(-0.2, 0.2, 4000)
    u = stb.potential_D(ctx, M, np.ones(4), pts, params=stb.default_params(n_g=n_g))
    ref = oracle.potential_dl(vtx, tet, normal, np.ones(4), pts, n_g=n_g)
    k = np.abs(ref) > 1e-3 * np.abs(ref).max()
    assert k.sum() > 3000
    assert np.quantile(np.abs(u[k] - ref[k]) / np.abs(ref[k]), 0.7) <= 24 * 2.0 ** -53
    M.close()


# fewer nodes than a piece's lanes, one more, and two rounds of them; points whose
# cones meet a panel's plane in whole circles (no breakpoints) and in short pieces;
# one workgroup's share of every job list and several
@pytest.mark.parametrize("n_g", [2, 15, 17, 33])
@pytest.mark.parametrize("slabs", [1, 4])
def test_full_evaluation_nodes(stb, ctx, n_g, slabs):
    mesh = inputs.icosphere_mesh(0, slabs, T=float(slabs))
    M = stb.Mesh(ctx, mesh.vtx, mesh.tets)
    M.set_normals(mesh.outward_normals())
    v = np.random.default_rng(4).standard_normal(mesh.nv)
    cen = mesh.tet_coords().mean(axis=1)
    off = np.concatenate([np.full((len(cen), 1), 0.05), 1e-3 * mesh.outward_normals()], axis=1)
    pts = np.concatenate([cen + off, cen + [0.2, 1e-3, 0, 0], inputs.shell_points(40, mesh.T, seed=9)])
    u = stb.potential_D(ctx, M, v, pts, params=stb.default_params(n_g=n_g))
    ref = oracle.potential_dl(mesh.vtx, mesh.tets, mesh.outward_normals(), v, pts, n_g=n_g)
    # the double layer's parity bound
    assert np.all(np.abs(u - ref) <= 1e-10 * np.maximum(np.abs(ref), 1e-5 * np.abs(ref).max()))
    M.close()
