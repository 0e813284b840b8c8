"""GPU tests of calls at the limits of what the library takes: values that are not finite, the largest launches,
memory that a call may need, and which launch shapes and paths a call leaves behind."""
import numpy as np
import pytest
import scipy.special as sp
import torch

import oracle
from paper_1908_07392_amd import mhlp
from paper_1908_07392_amd import workloads as wl

pytestmark = pytest.mark.gpu


def _t(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device="cuda:0")


@pytest.mark.parametrize("px,py", [(np.inf, None), (-np.inf, None), (None, -np.inf), (np.inf, np.inf), (np.inf, np.nan)])
def test_volume_points_at_infinity(px, py):
    """A point at infinity keeps its cluster from being left out of any sum: the values that are not finite are those
    of the sum over all pairs, and the others agree with it."""
    rng = np.random.default_rng(1)
    n, alpha, h = 13000, 12.0, 0.01
    x, y = rng.uniform(-1.5, 1.5, n), rng.uniform(-1.5, 1.5, n)
    x[4321] = x[4321] if px is None else px
    y[4321] = y[4321] if py is None else py
    w, f = np.full(n, 1.0 / n), rng.standard_normal(n)
    out = torch.empty(n, dtype=torch.float64, device="cuda:0")
    u = mhlp.volume_eval(_t(x), _t(y), _t(w), _t(f), alpha, h)[0].cpu().numpy()
    v = mhlp.volume_eval_noalloc(_t(x), _t(y), _t(w), _t(f), alpha, h, out).cpu().numpy()
    assert np.array_equal(np.isnan(u), np.isnan(v)) and np.array_equal(np.isposinf(u), np.isposinf(v))
    ok = np.isfinite(v)
    assert (np.abs(u[ok] - v[ok]) <= 1e-12 * np.abs(v[ok]).max(initial=0.0)).all()


@pytest.mark.parametrize("sign", [1.0, -1.0])
def test_opposite_infinities_near_and_far(sign):
    """A plan whose far items may be left out, an infinite charge near a group of targets and the opposite one far from
    it: every pair of both has K0 > 0, so the sum is NaN at every target, and with one of them alone it is infinite."""
    rng = np.random.default_rng(3)
    m, alpha = 41000, 150.0
    g = wl.discretize(wl.Curve("ellipse", a=1.2, b=0.7), 40)
    # targets within 4.3 of every node (z < 650, above the underflow) and away from the near panels
    tx, ty = rng.uniform(-2.4, 2.4, 3 * m), rng.uniform(-1.6, 1.6, 3 * m)
    clear = 1.3 * g.weights.reshape(-1, 16).sum(axis=1).max()
    far = np.ones(3 * m, bool)
    for j in range(0, g.n_nodes, 3):
        far &= np.hypot(tx - g.x[j], ty - g.y[j]) > clear
    tx, ty = tx[far][:m], ty[far][:m]
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    assert P.n_targets == m and P.n_near_pairs == 0
    left, right = int(np.argmin(g.x)), int(np.argmax(g.x))
    for bad in ((left,), (right,), (left, right)):
        sg = rng.standard_normal(g.n_nodes)
        for k, j in enumerate(bad):
            sg[j] = sign * np.inf * (-1) ** k
        u = mhlp.eval_slp(P, _t(sg)).cpu().numpy()
        assert np.isnan(u).all() if len(bad) == 2 else (u == sign * np.inf).all()


def test_gemm_of_more_tiles_than_a_grid_dimension_holds():
    """131,072 x 131,072 from one column and one row (4096^2 tiles of 256 threads: 2^32 threads); products of small
    whole numbers are exact."""
    n = 131072
    if torch.cuda.mem_get_info()[0] < 80 << 30:
        pytest.skip("needs 69 GB for the product")
    a = torch.arange(n, device="cuda:0") % 13 - 6
    b = torch.arange(n, device="cuda:0") % 7 - 3
    c = mhlp.gemm_bf16(a.float()[:, None].contiguous(), b.float()[None, :].contiguous())
    for i in (0, 31, 32, 65535, 65536, n - 33, n - 1):
        assert torch.equal(c[i], (a[i] * b).float()) and torch.equal(c[:, i], (a * b[i]).float())


def test_box_values_at_more_points_than_a_grid_dimension_holds():
    """2^28 + 5 points, 16 lanes each: the first and last ones as in a small call."""
    n = (1 << 28) + 5
    if torch.cuda.mem_get_info()[0] < 16 << 30:
        pytest.skip("needs 9 GB for the points and values")
    M = 16
    B = mhlp.Box(M, -1.0, 0.5, 2.0, 3.0)
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    F = torch.randn(2, M, M, dtype=torch.float64, device="cuda:0", generator=gen)
    px = torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen)
    py = torch.rand(n, dtype=torch.float64, device="cuda:0", generator=gen)
    up = B.particular(F, want_u=False, px=px, py=py)[2]
    for cut in (slice(0, 1000), slice(n - 1000, n)):
        small = B.particular(F, want_u=False, px=px[cut].clone(), py=py[cut].clone())[2]
        assert torch.equal(up[:, cut], small)


def test_network_workspace_does_not_grow_with_the_batch():
    """Besides the seven activation buffers of a network (batch x its widest layer) a training step allocates the
    partial tiles of its split products, which stay below 2 x 512 tiles of 4 KB."""
    batch, wide = 32768, 256
    N = mhlp.MLP(64, wide, wide, seed=3)
    X, T = torch.randn(batch, 64, device="cuda:0"), torch.randn(batch, wide, device="cuda:0")
    N.loss_grad(X[:16], T[:16])  # code and torch's own buffers in place
    N.loss_grad(X[:16].clone(), T[:16].clone())
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    N.loss_grad(X, T)
    torch.cuda.synchronize()
    assert free - torch.cuda.mem_get_info()[0] <= 7 * batch * wide * 4 + (64 << 20)


def test_tuning_launches_without_a_split_leaves_it():
    """The gradients and the stresslet do not use a plan's source split: tuning them keeps the one that shapes the
    plan's mixed-precision launches, whether timed or asked of the cache."""
    from paper_1908_07392_amd import autotune
    g = wl.discretize(wl.starfish_curve(), 64)
    G = mhlp.Geometry(_t(g.node_soa()))
    tx, ty = (_t(v) for v in wl.grid_targets(60, -0.6, 0.6))
    for stokes, layers in ((False, ("grad",)), (True, ("stokes", "stokes_grad"))):
        P = mhlp.Plan(G, 20.0, tx, ty, stokes=stokes)
        for split in (16, 32):
            P.set_split(split)
            for name in layers:
                best, ms, table = P.autotune(layers=autotune.LAYERS[name], reps=1)
                assert best == P.nsplit == split and list(table) == [split] and ms == table[split]
                assert autotune.tune(P, name, reps=1)["nsplit"] == P.nsplit == split


def test_batch_shapes_of_one_launch_share_a_time():
    g = wl.discretize(wl.starfish_curve(), 40)
    B = mhlp.Batch([mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 9.0)], 2)
    B.autotune(reps=2)
    rows = B.tile()["candidates"]
    for target in {r[0] for r in rows}:
        same = [r for r in rows if r[0] == target]
        assert len(same) == 4 and len({r[3] for r in same}) == 1


@pytest.mark.parametrize("alpha", [5.0, 200.0])
def test_mixed_solve_is_the_fp64_solve(alpha):
    """The operator is FP64 in both precisions, so a mixed-precision solve takes the same single cycle."""
    g = wl.discretize(wl.starfish_curve(), 96)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha)
    b = _t(np.cos(3 * g.theta) + 0.5)
    mu64, i64 = mhlp.gmres_solve(P, b, tol=1e-10)
    mu32, i32 = mhlp.gmres_solve(P, b, tol=1e-10, precision=mhlp.MIXED)
    assert i64 == i32 and i32["converged"] and torch.equal(mu64, mu32)


@pytest.mark.parametrize("alpha", [0.05, 5.0, 50.0, 500.0])
def test_fmm_at_a_level_that_the_caller_asks_for(alpha):
    """An explicit leaf level is served by the FMM whatever the lists would take: not the lists' values bit for bit,
    yet as near to the oracle's (1e-11) and to theirs (1e-12) as the FMM's own tests ask, from level 0 to the finest."""
    curve = wl.starfish_curve()
    g = wl.discretize(curve, 128)
    rng = np.random.default_rng(int(alpha * 100) + 9)
    th = rng.uniform(0, 2 * np.pi, 60)
    z, dz, _ = curve.eval(th)
    pts = np.concatenate([z + d * 1j * dz / np.abs(dz) for d in (3e-2, 1e-4, -1e-3)] +
                         [rng.uniform(-1.6, 1.6, 300) + 1j * rng.uniform(-1.6, 1.6, 300)])
    mu = wl.fourier_density(g.theta, wl.random_fourier_coeffs(rng, 8))
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(pts.real), _t(pts.imag))
    lists = mhlp.eval_layer(P, sigma=_t(mu), mu=_t(mu))
    exact = oracle.eval_potentials(g.x, g.y, alpha, pts.real, pts.imag, sigma=mu, mu=mu)
    P.set_fmm(40)
    for level in range(P.fmm[1] + 1):
        P.set_fmm(40, level)
        for u, v, w in zip(mhlp.eval_layer(P, sigma=_t(mu), mu=_t(mu)), lists, exact):
            assert not torch.equal(u, v) and float((u - v).abs().max()) < 1e-12 * float(v.abs().max())
            assert np.max(np.abs(u.cpu().numpy() - w)) < 1e-11 * np.max(np.abs(w))


def test_lists_take_the_memory_of_their_items():
    """A million targets and 2048 panels at small alpha: the lists hold a few hundred items a group, not an entry a
    panel (256 MB), and are built in several parts.  The values are those of the same targets in a small plan: each
    good to about 30 roundings of the sum of absolute values, which for these positive terms is the value."""
    g = wl.discretize(wl.starfish_curve(), 2048)
    G = mhlp.Geometry(_t(g.node_soa()))
    tx, ty = (_t(v) for v in wl.grid_targets(1000, -1.7, 1.7))
    mhlp.Plan(G, 3.0, tx, ty)  # the runtime's own memory for these launches is in place after it
    torch.cuda.synchronize()
    free = torch.cuda.mem_get_info()[0]
    P = mhlp.Plan(G, 3.0, tx, ty)
    torch.cuda.synchronize()
    near = P.n_near_pairs * (2 * 16 * 8 + 24)
    # 96 MB of partial sums and 32 MB of classes of the mixed tiles, 40 MB of targets and their lists' places
    assert free - torch.cuda.mem_get_info()[0] < near + (256 << 20)
    u = mhlp.eval_slp(P, _t(np.cos(3 * g.theta) + 1.5))
    pick = torch.randint(0, tx.numel(), (3000,), device="cuda:0", generator=torch.Generator("cuda:0").manual_seed(1))
    v = mhlp.eval_slp(mhlp.Plan(G, 3.0, tx[pick].clone(), ty[pick].clone()), _t(np.cos(3 * g.theta) + 1.5))
    assert float(((u[pick] - v) / v).abs().max()) < 1e-13


@pytest.mark.parametrize("stokes", [False, True])
def test_plan_without_memory_for_its_lists(stokes):
    """With memory left for what a plan holds but not for building its lists beside it, the plan still comes about,
    its pairs summed one by one: the values of the plan with lists (for the scalar alpha all its items are pairs, too)
    to the roundings of 16,384 terms."""
    g = wl.discretize(wl.starfish_curve(), 1024)
    G = mhlp.Geometry(_t(g.node_soa()))
    alpha, rng = (1e-5, 4.0)[stokes], np.random.default_rng(8)
    tx, ty = _t(rng.uniform(-1.5, 1.5, 300000)), _t(rng.uniform(-1.5, 1.5, 300000))
    mu = _t(np.stack([np.cos(3 * g.theta) + 1.5, np.sin(g.theta)])) if stokes else _t(np.cos(3 * g.theta) + 1.5)
    run = mhlp.stokes_eval if stokes else mhlp.eval_slp
    want = run(mhlp.Plan(G, alpha, tx, ty, stokes=stokes), mu)
    torch.cuda.synchronize()
    torch.cuda.empty_cache()
    free = torch.cuda.mem_get_info()[0]
    P = mhlp.Plan(G, alpha, tx, ty, stokes=stokes)
    torch.cuda.synchronize()
    holds = free - torch.cuda.mem_get_info()[0]
    del P
    # the lists pass through slots of 40 MB
    rest = torch.empty(torch.cuda.mem_get_info()[0] - holds - (10 << 20), dtype=torch.uint8, device="cuda:0")
    try:
        P = mhlp.Plan(G, alpha, tx, ty, stokes=stokes)
    finally:
        del rest
        torch.cuda.empty_cache()
    got = run(P, mu)
    assert float((got - want).abs().max()) < 1e-12 * float(want.abs().max())


@pytest.mark.parametrize("panels,alpha", [(300, 500.0), (600, 900.0), (257, 300.0)])
def test_items_left_out_on_the_curve(panels, alpha):
    """cos(n theta) is an eigenfunction of 1/2 I + D on the circle, with -alpha I_n K_n', on plans whose operator
    leaves far items out (one block a group, a large spread of z); a density that lives on one panel leaves the far
    targets what the far items bring: there the panel's plain sum."""
    g = wl.discretize(wl.Curve("circle", R=1.0), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha)
    lam = -alpha * sp.ive(2, alpha) * np.exp(alpha) * sp.kvp(2, alpha) if alpha < 700 else None
    mu = np.cos(2 * g.theta)
    if lam is not None:
        out = mhlp.apply_bie(P, _t(mu)).cpu().numpy()
        assert np.max(np.abs(out - lam * mu)) < 1e-11 * abs(lam)
    one = np.zeros(g.n_nodes)
    one[16 * 40:16 * 41] = 1.0 + np.arange(16) / 7.0
    out = mhlp.apply_bie(P, _t(one)).cpu().numpy()
    k = np.arange(g.n_nodes)
    far = np.minimum(np.abs(k - 648), g.n_nodes - np.abs(k - 648)) > 16 * 6
    ex, ey = g.x[far][:, None] - g.x[16 * 40:16 * 41], g.y[far][:, None] - g.y[16 * 40:16 * 41]
    r = np.hypot(ex, ey)
    nx, ny = (n[16 * 40:16 * 41] for n in g.normals)
    size = alpha * sp.k1(alpha * r) / (2 * np.pi) * (g.weights * one)[16 * 40:16 * 41]
    d = size / r * (ex * nx + ey * ny)
    assert (np.abs(out[far] - d.sum(axis=1)) <= ((3e-14 + 5e-16 * alpha * r) * size).sum(axis=1) + 1e-300).all()


@pytest.mark.parametrize("panels,m", [(16, 60), (64, 300), (256, 60), (64, 960), (64, 2500), (50, 5000), (40, 9000),
                                      (64, 20000)])
def test_split_groups_finish_alike(panels, m):
    """Groups summed by several blocks, the last of which adds the slots: the same bits whichever that is, in calls
    of either layer, gradients and both in turn, and in replays of a captured graph between them."""
    g = wl.discretize(wl.starfish_curve(), panels)
    rng = np.random.default_rng(m)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 15.0, _t(rng.uniform(-1.5, 1.5, m)), _t(rng.uniform(-1.5, 1.5, m)))
    sg = _t(np.cos(3 * g.theta) + 0.5)
    first = [mhlp.eval_slp(P, sg), *mhlp.eval_layer(P, sigma=sg, mu=sg), *mhlp.eval_grad(P, sigma=sg, mu=sg)]
    assert torch.equal(first[0], first[1])  # one layer alone as beside the other
    out = torch.empty_like(first[0])
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.stream(side), torch.cuda.graph(graph, stream=side):
        mhlp.eval_slp(P, sg, out=out)
    torch.cuda.synchronize()
    for k in range(20):
        out.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, first[0])
        again = [mhlp.eval_slp(P, sg), *mhlp.eval_layer(P, sigma=sg, mu=sg), *mhlp.eval_grad(P, sigma=sg, mu=sg)]
        assert all(torch.equal(a, b) for a, b in zip(first, again))


@pytest.mark.parametrize("panels,m", [(16, 1), (16, 64 * 64), (17, 64 * 63), (64, 64 * 16), (63, 64 * 16 + 1),
                                      (40, 26000), (40, 27000)])
def test_small_plans_summed_pair_by_pair(panels, m):
    """Plans on both sides of the sizes up to which all pairs are summed and charges are formed where they are read:
    each of the potentials, gradients and the stresslet as the same targets give beside others in a larger plan with
    expansions (which the plain sums of their own tests check): 30 roundings of the sum of absolute values, here the
    largest value times 1e-12."""
    g = wl.discretize(wl.starfish_curve(), panels)
    rng = np.random.default_rng(m)
    G = mhlp.Geometry(_t(g.node_soa()))
    k = max(m, 30000)
    tx, ty = rng.uniform(-1.5, 1.5, k), rng.uniform(-1.5, 1.5, k)
    mu = _t(np.cos(3 * g.theta) + 0.5)
    mu2 = _t(np.stack([np.cos(2 * g.theta), np.sin(g.theta)]))
    for alpha in (2.0, 150.0):
        small, large = (mhlp.Plan(G, alpha, _t(tx[:n]), _t(ty[:n])) for n in (m, k))
        got = [*mhlp.eval_layer(small, sigma=mu, mu=mu), mhlp.eval_slp(small, mu), mhlp.eval_dlp(small, mu),
               *mhlp.eval_grad(small, sigma=mu, mu=mu), mhlp.eval_grad(small, sigma=mu)[0], mhlp.eval_grad(small, mu=mu)[1]]
        want = [*mhlp.eval_layer(large, sigma=mu, mu=mu), mhlp.eval_slp(large, mu), mhlp.eval_dlp(large, mu),
                *mhlp.eval_grad(large, sigma=mu, mu=mu), mhlp.eval_grad(large, sigma=mu)[0], mhlp.eval_grad(large, mu=mu)[1]]
        small, large = (mhlp.Plan(G, alpha, _t(tx[:n]), _t(ty[:n]), stokes=True) for n in (m, k))
        got += [mhlp.stokes_eval(small, mu2), mhlp.stokes_eval_grad(small, mu2)]
        want += [mhlp.stokes_eval(large, mu2), mhlp.stokes_eval_grad(large, mu2)]
        for a, b in zip(got, want):
            assert float((a - b[..., :m]).abs().max()) <= 1e-12 * float(b.abs().max())


@pytest.mark.parametrize("bad", [float("nan"), float("inf"), -float("inf")])
def test_non_finite_densities_of_small_plans(bad):
    """As in larger plans: a NaN or infinite charge or dipole reaches every target, also where its pairs underflow."""
    g = wl.discretize(wl.starfish_curve(), 20)
    rng = np.random.default_rng(2)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 900.0, _t(rng.uniform(-1.5, 1.5, 500)), _t(rng.uniform(-1.5, 1.5, 500)))
    v = np.ones(g.n_nodes)
    v[77] = bad
    for u in (mhlp.eval_slp(P, _t(v)), mhlp.eval_dlp(P, _t(v)), *mhlp.eval_grad(P, sigma=_t(v), mu=_t(v))):
        assert not torch.isfinite(u).any()


@pytest.mark.parametrize("alpha,fmm", [(20.0, False), (1000.0, True)])
def test_automatic_choice_at_large_alpha(alpha, fmm):
    """Where the boxes' neighbours underflow the FMM has little left to do and serves (49,729 points, 256 panels:
    59 us against 98); at smaller alpha the lists do."""
    g = wl.discretize(wl.starfish_curve(), 256)
    tx, ty = wl.grid_targets(223, -1.4, 1.4)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha, _t(tx), _t(ty))
    mu = _t(np.cos(3 * g.theta) + 0.5)
    lists = mhlp.eval_slp(P, mu)
    P.set_fmm(40)
    u = mhlp.eval_slp(P, mu)
    assert torch.equal(u, lists) != fmm and float((u - lists).abs().max()) < 1e-12 * float(lists.abs().max())


@pytest.mark.parametrize("groups", [40, 41, 61, 62, 327, 328])
def test_charges_formed_where_read_or_staged(groups):
    """Plans without expansions on both sides of the sizes up to which charges are formed where they are read, which
    depend on the layers: the single layer, and the double layer's gradient, have the same bits alone as beside the
    other (a double layer alone rounds K1 otherwise, as it needs no K0)."""
    g = wl.discretize(wl.starfish_curve(), 50)
    rng = np.random.default_rng(groups)
    m = 64 * groups
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 95.0, _t(rng.uniform(-1.6, 1.6, m)), _t(rng.uniform(-1.6, 1.6, m)))
    sg, mu = _t(np.cos(3 * g.theta) + 0.5), _t(np.sin(2 * g.theta) + 0.25)
    assert torch.equal(mhlp.eval_slp(P, sg), mhlp.eval_layer(P, sigma=sg, mu=mu)[0])
    assert torch.equal(mhlp.eval_grad(P, mu=mu)[1], mhlp.eval_grad(P, sigma=sg, mu=mu)[1])


@pytest.mark.parametrize("panels", [16, 70, 139, 341, 344])
def test_operator_of_any_number_of_blocks_a_group(panels):
    """cos(2 theta) is an eigenfunction of 1/2 I + D on the circle, with -alpha I_n K_n', where a group's blocks are as
    many as fill the chip: the same bits each time, and within 1e-11 of it."""
    g = wl.discretize(wl.Curve("circle", R=1.0), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), 20.0)
    lam = -20.0 * sp.iv(2, 20.0) * sp.kvp(2, 20.0)
    mu = np.cos(2 * g.theta)
    first = mhlp.apply_bie(P, _t(mu))
    for k in range(20):
        assert torch.equal(mhlp.apply_bie(P, _t(mu)), first)
    assert np.max(np.abs(first.cpu().numpy() - lam * mu)) < 1e-11 * abs(lam)


@pytest.mark.parametrize("panels,alpha", [(198, 200.0), (256, 500.0), (360, 350.0), (700, 500.0)])
def test_items_left_out_beside_tiny_sums(panels, alpha):
    """On the curve, a density over 260 decades: where it is tiny, the items of the panels where it is not have to be
    summed, whatever the nearest ones give.  The kernel has one sign on the circle, so that the values of the loud and
    the quiet part of the density add up to those of the whole to 1e-12 at every node (left out: 2^-55)."""
    g = wl.discretize(wl.Curve("circle", R=1.0), panels)
    P = mhlp.Plan(mhlp.Geometry(_t(g.node_soa())), alpha)
    mu = np.exp(-600.0 * np.sin(g.theta / 2) ** 2)
    loud = np.where(mu > 1e-20, mu, 0.0)
    whole, again, a, b = (mhlp.eval_dlp(P, _t(v)) for v in (mu, mu, loud, mu - loud))
    assert torch.equal(whole, again)
    assert bool(torch.all(torch.abs(whole - a - b) <= 1e-12 * torch.abs(whole)))
