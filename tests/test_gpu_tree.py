"""GPU tests of the cluster-expansion far field (csrc/tree.h) at the sizes where its lists and splits can
go wrong: ragged clusters, one target to many, every regime of alpha R.

Off the near panels the result is the plain Nystrom sum, which scipy's K0 and K1 give pair by pair.  The
bound of a term is 3e-14 + 5e-16 z of its absolute value: about 10 roundings of 2.2e-16 per term and
partial sum, times the spread of the kernel over a cluster (I0(2) = 2.3 on average over its charges),
with a margin of six, and two roundings of the argument of e^{-z} on either side; 1e-300 covers values next
to underflow.  In mixed precision a term is
good to 1e-6 plus 2e-7 z (three roundings of 2^-24 in the argument of e^{-z}); below 1e-36 of the charges
it is flushed to zero."""
import numpy as np
import pytest
import scipy.special as sp
import torch

from paper_1908_07392_amd import mhlp
from paper_1908_07392_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


def _setup(panels, m, seed):
    """An ellipse, random densities, targets inside and outside further than 1.25 panel lengths from it."""
    rng = np.random.default_rng(seed)
    g = wl.discretize(wl.Curve("ellipse", a=1.2, b=0.7), panels)
    clear = 1.3 * g.weights.reshape(-1, 16).sum(axis=1).max()
    tx, ty = rng.uniform(-3.0, 3.0, 40 * m + 400), rng.uniform(-2.0, 2.0, 40 * m + 400)
    tx[: tx.size // 2] *= 0.3
    ty[: ty.size // 2] *= 0.3
    keep = np.ones(tx.size, bool)
    for j in range(0, g.n_nodes, 3):
        keep &= np.hypot(tx - g.x[j], ty - g.y[j]) > clear
    tx, ty = tx[keep], ty[keep]
    pick = rng.permutation(tx.size)[:m]
    assert pick.size == m
    return g, tx[pick], ty[pick], rng.standard_normal(g.n_nodes), rng.standard_normal(g.n_nodes)


def _plain(g, alpha, tx, ty, sg, mu):
    """The sums, and the sums of the terms' absolute values times the FP64 and the mixed bound of a term."""
    ex, ey = tx[:, None] - g.x, ty[:, None] - g.y
    r = np.hypot(ex, ey)
    nx, ny = g.normals
    s = sp.k0(alpha * r) * (g.weights * sg) / (2 * np.pi)
    d = alpha * sp.k1(alpha * r) / r * (ex * nx + ey * ny) * (g.weights * mu) / (2 * np.pi)
    dabs = alpha * sp.k1(alpha * r) * np.abs(g.weights * mu) / (2 * np.pi)
    f64, f32 = 3e-14 + 5e-16 * alpha * r, 1e-6 + 2e-7 * alpha * r
    return (s.sum(axis=1), (np.abs(s) * f64).sum(axis=1), (np.abs(s) * f32).sum(axis=1),
            d.sum(axis=1), (dabs * f64).sum(axis=1), (dabs * f32).sum(axis=1))


# alpha R of a panel from 1e-7 (below the expansions' range: all direct) through the expansions to beyond
# them; at 900 the farthest pairs underflow.  Target counts on both sides of a group of 64 and of every
# split of the groups over waves and blocks.
@pytest.mark.parametrize("panels,m,alpha", [(24, 1, 3.0), (40, 63, 1e-6), (40, 65, 0.05), (47, 64, 3.0), (33, 1000, 8.0),
                                            (64, 5500, 20.0), (31, 11000, 60.0), (40, 41000, 12.0), (48, 300, 900.0),
                                            (37, 77000, 2.0)])
def test_tree_potentials_vs_plain_sums(panels, m, alpha):
    g, tx, ty, sg, mu = _setup(panels, m, panels + m)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    assert P.n_near_pairs == 0
    sel = np.unique(np.linspace(0, m - 1, min(m, 400)).astype(int))
    s, sa, sm, d, da, dm = _plain(g, alpha, tx[sel], ty[sel], sg, mu)
    for prec in (mhlp.FP64, mhlp.MIXED):
        us, ud = mhlp.eval_layer(P, sigma=_t(sg), mu=_t(mu), precision=prec)
        us1, ud1 = mhlp.eval_slp(P, _t(sg), precision=prec), mhlp.eval_dlp(P, _t(mu), precision=prec)
        for u, ref, a64, a32 in ((us, s, sa, sm), (us1, s, sa, sm), (ud, d, da, dm), (ud1, d, da, dm)):
            bound = a64 + 1e-300 if prec == mhlp.FP64 else a32 + 1e-36 * alpha
            assert (np.abs(u.cpu().numpy()[sel] - ref) <= bound).all()


def test_tree_clusters_leave_listed_panels_direct():
    """A near factor that lists panels far from their targets: no cluster may cover a listed panel.  On a
    resolved curve with a smooth density the corrected panels give the plain rule's value."""
    g, tx, ty, _, _ = _setup(96, 700, 5)
    sg = np.cos(3 * g.theta) + 0.5
    G = mhlp.Geometry(_t(g.node_soa()))
    plain = mhlp.Plan(G, 6.0, _t(tx), _t(ty))
    wide = mhlp.Plan(G, 6.0, _t(tx), _t(ty), params=dict(near_factor=9.0, rho_direct=200.0))
    assert plain.n_near_pairs == 0 and wide.n_near_pairs > 700
    for a, b in zip(mhlp.eval_layer(plain, sigma=_t(sg), mu=_t(sg)), mhlp.eval_layer(wide, sigma=_t(sg), mu=_t(sg))):
        assert float((a - b).abs().max()) < 1e-9 * float(a.abs().max())


@pytest.mark.parametrize("alpha", [5.0, 900.0])
@pytest.mark.parametrize("bad", [float("nan"), float("inf")])
def test_tree_non_finite_densities_reach_every_target(alpha, bad):
    """A NaN or infinite charge makes every target non-finite, also where its pairs underflow; an infinite
    one gives +inf wherever K0 is not zero, as the sum pair by pair does."""
    g, tx, ty, sg, _ = _setup(48, 300, 7)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    sg[100] = bad
    u = mhlp.eval_slp(P, _t(sg)).cpu().numpy()
    if np.isnan(bad):
        assert np.isnan(u).all()
    else:
        z = alpha * np.hypot(tx - g.x[100], ty - g.y[100])
        assert (u[z < 700.0] == np.inf).all() and not np.isfinite(u).any()


@pytest.mark.parametrize("panels", [3, 17, 96, 170, 700])
@pytest.mark.parametrize("alpha", [2.0, 40.0])
def test_tree_onsurface_operator_on_the_circle(panels, alpha):
    """cos(n theta) is an eigenfunction of 1/2 I + D on the circle, with -alpha I_n K_n'."""
    g = wl.discretize(wl.Curve("circle", R=1.0), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha)
    n = 2
    lam = -alpha * sp.ive(n, alpha) * np.exp(alpha) * sp.kvp(n, alpha)
    mu = np.cos(n * g.theta)
    for prec, tol in ((mhlp.FP64, 1e-11 if panels > 3 else 1e-6), (mhlp.MIXED, 1e-6)):
        out = mhlp.apply_bie(P, _t(mu), precision=prec).cpu().numpy()
        assert np.max(np.abs(out - lam * mu)) < tol * abs(lam)


@pytest.mark.parametrize("panels,m,alpha", [(29, 1, 4.0), (33, 900, 8.0), (64, 5500, 25.0), (31, 11000, 60.0),
                                            (40, 41000, 3.0), (37, 77000, 12.0)])
def test_tree_gradients_vs_plain_sums(panels, m, alpha):
    """Each component against the closed forms, to the potentials' bound times alpha (the size of a derivative)
    and the dipole's second derivative."""
    g, tx, ty, sg, mu = _setup(panels, m, panels + m)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    sel = np.unique(np.linspace(0, m - 1, min(m, 400)).astype(int))
    ex, ey = tx[sel][:, None] - g.x, ty[sel][:, None] - g.y
    r = np.hypot(ex, ey)
    k0, k1 = sp.k0(alpha * r), sp.k1(alpha * r)
    nx, ny = g.normals
    q, d = g.weights * sg / (2 * np.pi), g.weights * mu / (2 * np.pi)
    A, f64 = alpha * k1 / r, 3e-14 + 5e-16 * alpha * r
    B = (ex * nx + ey * ny) * (alpha ** 2 * k0 + 2 * A) / r ** 2
    gs, gd = mhlp.eval_grad(P, sigma=_t(sg), mu=_t(mu))
    gs1, gd1 = mhlp.eval_grad(P, sigma=_t(sg))[0], mhlp.eval_grad(P, mu=_t(mu))[1]
    for u, v in ((gs, gd), (gs1, gd1)):
        for c, (e, n) in enumerate(((ex, nx), (ey, ny))):
            bs = (A * r * np.abs(q) * f64).sum(axis=1)
            bd = ((alpha ** 2 * k0 + 3 * A) * np.abs(d) * f64).sum(axis=1)
            assert (np.abs(u[c].cpu().numpy()[sel] + (A * e * q).sum(axis=1)) <= bs + 1e-300).all()
            assert (np.abs(v[c].cpu().numpy()[sel] - ((A * n - B * e) * d).sum(axis=1)) <= bd + 1e-300).all()


def _stokeslets_T(alpha, r):
    z = alpha * r
    k0, zk1 = sp.k0(z), z * sp.k1(z)
    a1 = -(2 * z * z * k0 + (z * z + 4) * zk1 - 4) / (2 * np.pi * alpha ** 2 * r ** 4)
    a2 = (4 * z * z * k0 + (z * z + 8) * zk1 - 8) / (np.pi * alpha ** 2 * r ** 6)
    a3 = (zk1 - 1) / (2 * np.pi * r * r)
    return k0, zk1, a1, a2, a3


@pytest.mark.parametrize("panels,m,alpha", [(29, 1, 6.0), (33, 900, 12.0), (64, 5500, 25.0), (31, 11000, 60.0),
                                            (40, 41000, 9.0), (37, 77000, 300.0)])
def test_tree_stresslet_vs_plain_sums(panels, m, alpha):
    """Velocity and velocity gradient against the closed forms of App. B term by term.  Their brackets cancel
    like z^2/8, in the reference and in the expansions alike: a term's bound is the potentials' times
    1 + 16/z^2, of |m| 2/(pi r) for the velocity and of |m| 8/(pi r^2) for its derivatives."""
    g, tx, ty, m1, m2 = _setup(panels, m, panels + m)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty), stokes=True)
    mu = _t(np.stack([m1, m2]))
    sel = np.unique(np.linspace(0, m - 1, min(m, 300)).astype(int))
    e = [tx[sel][:, None] - g.x, ty[sel][:, None] - g.y]
    r = np.hypot(*e)
    n, d = g.normals, [g.weights * m1, g.weights * m2]
    k0, zk1, a1, a2, a3 = _stokeslets_T(alpha, r)
    rn, rm, nm = e[0] * n[0] + e[1] * n[1], e[0] * d[0] + e[1] * d[1], n[0] * d[0] + n[1] * d[1]
    size = np.hypot(*d) * (3e-14 + 5e-16 * alpha * r) * (1 + 16 / (alpha * r) ** 2)
    u = mhlp.stokes_eval(P, mu).cpu().numpy()
    for i in range(2):
        ref = -(a1 * (n[i] * rm + e[i] * nm + d[i] * rn) + (a2 * rm * rn + a3 * nm) * e[i]).sum(axis=1)
        assert (np.abs(u[i][sel] - ref) <= (2 / (np.pi * r) * size).sum(axis=1)).all()
    ak0 = alpha ** 2 * k0
    b1 = (ak0 / (2 * np.pi) - 4 * a1) / r ** 2
    b2 = -(ak0 + 2 * zk1 / r ** 2) / (np.pi * r ** 4) - 6 * a2 / r ** 2
    b3 = -(ak0 / (2 * np.pi) + 2 * a3) / r ** 2
    gr = mhlp.stokes_eval_grad(P, mu).cpu().numpy()
    for i in range(2):
        for l in range(2):
            p1 = n[i] * rm + e[i] * nm + d[i] * rn
            dp1 = n[i] * d[l] + (i == l) * nm + d[i] * n[l]
            dp2 = (i == l) * rm * rn + e[i] * (d[l] * rn + rm * n[l])
            ref = -(e[l] * (b1 * p1 + b2 * e[i] * rm * rn + b3 * e[i] * nm) + a1 * dp1 + a2 * dp2 +
                    a3 * (i == l) * nm).sum(axis=1)
            assert (np.abs(gr[i][l][sel] - ref) <= (8 / (np.pi * r * r) * size).sum(axis=1)).all()


@pytest.mark.parametrize("panels,alpha", [(3, 3.0), (17, 40.0), (170, 8.0), (300, 200.0)])
def test_tree_onsurface_stresslet_on_the_circle(panels, alpha):
    """(1/2 I + D + W) mu on the circle, at target counts that are no multiple of 64 and at every split: linear,
    and by rotational symmetry a multiple of n for mu = n."""
    g = wl.discretize(wl.Curve("circle", R=1.0), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, stokes=True)
    nx, ny = g.normals
    rng = np.random.default_rng(panels)
    c = rng.standard_normal(4)
    a = np.stack([np.cos(2 * g.theta), np.sin(3 * g.theta)])
    b = np.stack([nx, ny])
    A, B, AB = (mhlp.stokes_apply_bie(P, _t(v)).cpu().numpy() for v in (a, b, c[0] * a + c[1] * b))
    assert np.max(np.abs(AB - c[0] * A - c[1] * B)) < 1e-12 * (np.abs(A).max() + np.abs(B).max())
    tang = B[0] * ny - B[1] * nx
    norm = B[0] * nx + B[1] * ny
    tol = 1e-11 if panels > 3 else 1e-6
    assert np.max(np.abs(tang)) < tol and np.max(np.abs(norm - norm[0])) < tol


@pytest.mark.parametrize("panels,n_rhs", [((7, 70, 17, 33), 1), ((16, 8, 129), 2), ((65, 40, 6), 3), ((31, 90), 4),
                                          ((300,), 2), ((530, 9), 1)])
def test_batched_operator_and_solve_vs_single(panels, n_rhs):
    """The batched operator against each plan's own (the same lists, moments formed per right-hand side: 1e-12)
    and the lockstep solve against the single one: both stop at a relative residual of 1e-11 of a second-kind
    operator with a condition number below 100, so the solutions agree to 2e-9."""
    rng = np.random.default_rng(len(panels))
    plans = []
    for k, p in enumerate(panels):
        g = wl.discretize(wl.Curve("ellipse", a=1.2, b=0.7 + 0.1 * k), p)
        plans.append(mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 4.0 + 3.0 * k))
    B = mhlp.Batch(plans, n_rhs)
    systems = [(P, r) for P in plans for r in range(n_rhs)]
    mus = [_t(rng.standard_normal(P.geom.n_nodes)) for P, _ in systems]
    packed = B.pack(mus)
    single = [mhlp.apply_bie(P, mu) for (P, _), mu in zip(systems, mus)]
    for target in (1, 768, 1 << 14):
        B.set_tile(target)
        for got, want in zip(B.unpack(B.apply(packed)), single):
            assert float((got - want).abs().max()) <= 1e-12 * float(want.abs().max())
    rhs = [torch.cos((1 + r) * torch.arange(P.geom.n_nodes, device="cuda:0") * (2 * np.pi / P.geom.n_nodes))
           .double() for P, r in systems]
    sol, infos = B.gmres(B.pack(rhs), tol=1e-11, restart=40)
    for (P, _), b, got, info in zip(systems, rhs, B.unpack(sol), infos):
        want, _ = mhlp.gmres_solve(P, b, tol=1e-11, restart=40)
        assert info["converged"] and float((got - want).norm()) <= 2e-9 * float(want.norm())


def _volume_reference(x, y, q, alpha, sel):
    """Plain sums over all other points at the points `sel`, and the bounds of their errors."""
    r = np.hypot(x[sel][:, None] - x, y[sel][:, None] - y)
    same = r == 0.0
    k = np.where(same, 0.0, sp.k0(alpha * np.where(same, 1.0, r))) / (2 * np.pi)
    tol = ((3e-14 + 5e-16 * alpha * r) * k * np.abs(q)).sum(axis=1)
    return (k * q).sum(axis=1), tol + 1e-300 * np.abs(q).sum()


@pytest.mark.parametrize("n,alpha,shape", [(12288, 20.0, "square"), (12289, 3.0, "disc"), (13007, 100.0, "line"),
                                           (70001, 7.0, "square"), (20000, 900.0, "square"), (14000, 15.0, "heaps"),
                                           (12300, 40.0, "point"), (300000, 60.0, "square")])
def test_volume_by_clusters_vs_plain_sums(n, alpha, shape):
    """The volume sum at sizes around the tiles of its sort and lists: even and uneven distributions, points on a
    line, coincident points (left out of each other's sums), pairs that underflow."""
    rng = np.random.default_rng(n)
    x, y = rng.uniform(-1.5, 1.5, n), rng.uniform(-1.5, 1.5, n)
    if shape == "disc":
        a, r = rng.uniform(0, 2 * np.pi, n), np.sqrt(rng.uniform(0, 1, n))
        x, y = 1e-3 + r * np.cos(a), 5.0 + r * np.sin(a)
    elif shape == "line":
        y = 0.25 * x
    elif shape == "heaps":
        x, y = x.round(0) + 1e-3 * rng.standard_normal(n), y.round(0) + 1e-3 * rng.standard_normal(n)
        x[100:400], y[100:400] = x[0], y[0]
    elif shape == "point":
        x[:], y[:] = 0.3, -0.2
        x[::50] += 0.01
    w, f, h = rng.uniform(0.5, 1.5, n) / n, rng.standard_normal(n), 0.01
    u, wc = mhlp.volume_eval(_t(x), _t(y), _t(w), _t(f), alpha, h)
    u = u.cpu().numpy()
    sel = np.unique(np.linspace(0, n - 1, 200).astype(int))
    ref, tol = _volume_reference(x, y, w * f, alpha, sel)
    own = wc / h ** 2 * w[sel] * f[sel]
    assert (np.abs(u[sel] - ref - own) <= tol + 1e-14 * np.abs(own)).all()
    v, _ = mhlp.volume_eval(_t(x), _t(y), _t(w), _t(f), alpha, h)
    assert np.array_equal(u, v.cpu().numpy())


def test_volume_by_clusters_non_finite():
    """A non-finite charge or point reaches the values that it reaches in the sum over all pairs."""
    rng = np.random.default_rng(1)
    n, alpha, h = 13000, 12.0, 0.01
    x, y = rng.uniform(-1.5, 1.5, n), rng.uniform(-1.5, 1.5, n)
    w, f = np.full(n, 1.0 / n), rng.standard_normal(n)
    out = torch.empty(n, dtype=torch.float64, device="cuda:0")
    for bad in ("charge", "point"):
        if bad == "charge":
            f[4000] = np.inf
        else:
            f[4000], x[17] = 0.5, np.nan
        u = mhlp.volume_eval(_t(x), _t(y), _t(w), _t(f), alpha, h)[0].cpu().numpy()
        v = mhlp.volume_eval_noalloc(_t(x), _t(y), _t(w), _t(f), alpha, h, out).cpu().numpy()
        assert np.array_equal(np.isnan(u), np.isnan(v)) and np.array_equal(np.isposinf(u), np.isposinf(v))
        assert not np.isfinite(u).any()


@pytest.mark.parametrize("alpha,order,fmm", [(5.0, 40, False), (200.0, 40, True), (200.0, 12, True)])
def test_fmm_or_lists(alpha, order, fmm):
    """set_fmm leaves FP64 evaluations to the cluster lists where those are shorter than the FMM's boxes (the same
    values, bit for bit), else the FMM serves: order 40 to rounding of the largest value (as the FMM's own tests),
    order 12 to its truncation, geometric from 1e-9 at order 20 (1e-5 with a margin)."""
    c = wl.Curve("starfish", R=1.0, A=0.3, k=5)
    g = wl.discretize(c, 896)
    q = np.linspace(-1.4, 1.4, 600)
    tx, ty = (v.ravel() for v in np.meshgrid(q, q))
    k = c.contains(tx, ty)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx[k]), _t(ty[k]))
    sigma, mu = _t(np.cos(3 * g.theta)), _t(np.sin(2 * g.theta))
    want = mhlp.eval_layer(P, sigma=sigma, mu=mu)
    P.set_fmm(order)
    assert P.fmm[0] == order
    got = mhlp.eval_layer(P, sigma=sigma, mu=mu) + (mhlp.eval_slp(P, sigma), mhlp.eval_dlp(P, mu))
    for a, b in zip(got, want + want):
        if fmm:
            assert not torch.equal(a, b)
            assert float((a - b).abs().max()) < (1e-12 if order == 40 else 1e-5) * float(b.abs().max())
        else:
            assert float((a - b).abs().max()) < 1e-13 * float(b.abs().max())
    if not fmm:
        assert torch.equal(got[0], want[0]) and torch.equal(got[1], want[1])


@pytest.mark.parametrize("panels,restart", [(200, 40), (257, 40), (520, 6), (1100, 60), (2100, 30)])
def test_gram_schmidt_over_slices(panels, restart):
    """Solves whose Gram-Schmidt runs over slices (every slice length, more than 64 of them, restarts): the residual
    formed by the operator itself meets the tolerance, with rounding of the two operator applications on top."""
    g = wl.discretize(wl.Curve("starfish", R=1.0, A=0.3, k=5), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 9.0)
    b = _t(np.cos(3 * g.theta) + np.where(np.arange(g.n_nodes) % 7 == 0, 0.5, 0.0))
    x, info = mhlp.gmres_solve(P, b, tol=1e-11, restart=restart)
    r = b - mhlp.apply_bie(P, x)
    assert info["converged"] and float(r.norm()) <= 1.1e-11 * float(b.norm()) + 1e-14 * float(x.norm())


@pytest.mark.parametrize("alpha,m", [(60.0, 41000), (400.0, 41000), (150.0, 77000)])
@pytest.mark.parametrize("density", ["one panel", "random", "small here, large there"])
def test_far_items_left_out_do_not_show(alpha, m, density):
    """Plans whose far items may be left out against the near ones' sum: where the near panels carry nothing or
    little, the far ones decide.  Bound as for every potential, per target."""
    g, tx, ty, sigma, mu = _setup(40, m, 7)
    if density == "one panel":
        keep = np.zeros(g.n_nodes)
        keep[16 * 5:16 * 6] = 1.0
        sigma, mu = sigma * keep, mu * keep
    elif density == "small here, large there":
        s = 10.0 ** (-60.0 * (0.5 + 0.5 * np.cos(g.theta)))
        sigma, mu = sigma * s, mu * s
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    us, ud = (v.cpu().numpy() for v in mhlp.eval_layer(P, sigma=_t(sigma), mu=_t(mu)))
    sel = np.unique(np.linspace(0, m - 1, 400).astype(int))
    dx, dy = tx[sel][:, None] - g.x, ty[sel][:, None] - g.y
    r = np.hypot(dx, dy)
    z = alpha * r
    ts = sp.k0(z) / (2 * np.pi) * g.weights * sigma
    nx, ny = g.normals
    td = alpha * sp.k1(z) / (2 * np.pi * r) * (dx * nx + dy * ny) * g.weights * mu
    size = alpha * sp.k1(z) / (2 * np.pi) * np.abs(g.weights * mu)
    tol = 3e-14 + 5e-16 * z
    assert (np.abs(us[sel] - ts.sum(axis=1)) <= (tol * np.abs(ts)).sum(axis=1) + 1e-300).all()
    assert (np.abs(ud[sel] - td.sum(axis=1)) <= (tol * size).sum(axis=1) + 1e-300).all()
