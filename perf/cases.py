"""Timed cases of the layer-potential framework, through its public entry points.

Every case has a "kind": one way in which a program uses the library.

  eval       layer potentials of given densities at the points of a grid inside the curve
  dirichlet  one boundary-value problem: GMRES for the density, then its potential at the grid
  grad       target gradients of both layers at the grid
  stokes     one modified-Stokes problem: GMRES on the 2N unknowns, then velocity and velocity gradient
  batch      boundary-value problems of many geometries at once, four right-hand sides each
  volume     the all-pairs volume sum on a tensor grid
  box        particular solution on a periodic box: grid values, gradient, values at boundary points
  train      one training step of the warm start's network: loss, gradient, Adam

`prepare` makes what a program holds before the call (geometry, plan, and the densities, data or forcing
that the seed draws), `run` is one pass, `exact` the same outputs in 64 bits from closed
forms, fine quadrature or plain torch.
"""
import math

import numpy as np
import torch

from paper_1908_07392_amd import mhlp
from paper_1908_07392_amd import workloads as wl

DEV = "cuda:0"
TWO_PI = 2.0 * math.pi
MARGIN = 2e-4  # relative distance of the targets from the curve, along the ray from its centre
MODES = 9      # Fourier modes of a density


def listed():
    """The sizes are those of the repository's benchmark and tests where it has them."""
    return [
        # one small evaluation, where the launches count: the circle of 64 panels with about 2800 targets
        {"name": "eval_circle_small", "kind": "eval", "curve": "circle", "panels": 64, "grid": 64, "alpha": 10.0,
         "layers": "both", "precision": "fp64", "fmm": 0},
        # the headline evaluation: starfish of 4096 nodes, about 109,000 targets, slow decay
        {"name": "eval_starfish_a5", "kind": "eval", "curve": "starfish", "panels": 256, "grid": 512, "alpha": 5.0,
         "layers": "both", "precision": "fp64", "fmm": 0},
        # the same curve at fast decay (small time steps), the double layer alone, a ragged target count
        {"name": "eval_starfish_a500_dlp", "kind": "eval", "curve": "starfish", "panels": 256, "grid": 487,
         "alpha": 500.0, "layers": "dlp", "precision": "fp64", "fmm": 0},
        # the FP32 far field that previews and inner solves take
        {"name": "eval_starfish_a50_mixed", "kind": "eval", "curve": "starfish", "panels": 256, "grid": 512,
         "alpha": 50.0, "layers": "both", "precision": "mixed", "fmm": 0},
        # the largest evaluation, where programs switch the fast multipole far field on
        {"name": "eval_fmm_large", "kind": "eval", "curve": "starfish", "panels": 896, "grid": 768, "alpha": 20.0,
         "layers": "both", "precision": "fp64", "fmm": 40},
        # a whole Dirichlet solve to 1e-10 and its solution on a coarse grid: one implicit step of a scalar problem
        {"name": "dirichlet_starfish_a5", "kind": "dirichlet", "curve": "starfish", "panels": 256, "grid": 128,
         "alpha": 5.0, "precision": "fp64"},
        # post-processing: both gradients at every point of the headline grid
        {"name": "grad_starfish_a50", "kind": "grad", "curve": "starfish", "panels": 256, "grid": 512, "alpha": 50.0},
        # a whole modified-Stokes step's boundary part, with velocity and velocity gradient inside
        {"name": "stokes_starfish_a50", "kind": "stokes", "curve": "starfish", "panels": 256, "grid": 256,
         "alpha": 50.0},
        # many small systems at once: 16 curves of 32 to 160 panels, alpha over three decades, 64 systems
        {"name": "batch_16x4", "kind": "batch", "geometries": 16, "panels_lo": 32, "panels_hi": 160, "mix": 4},
        # the dense stress case: 256 x 256 points, 4.3e9 pairs
        {"name": "volume_256", "kind": "volume", "n": 256, "alpha": 20.0, "precision": "fp64"},
        # the Fourier part of an implicit step: 512 x 512 box with gradient and 4096 boundary points
        {"name": "box_512", "kind": "box", "M": 512, "points": 4096, "alpha": 50.0},
        # one step of the warm start's training: 96 windows, 4096 -> 256 -> 256 -> 1024
        {"name": "train_96", "kind": "train", "batch": 96, "n_in": 4096, "width": 256, "n_out": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi + 0.49)))))


def _log(rng, lo, hi):
    return round(math.exp(rng.uniform(math.log(lo), math.log(hi))), 3)


def draw(rng):
    """A case of the same kinds and ranges; odd sizes as they come."""
    kind = rng.choice(["eval", "eval", "eval", "dirichlet", "grad", "stokes", "batch", "volume", "box", "train"])
    if kind == "eval":
        fmm = rng.random() < 0.2
        return {"kind": kind, "curve": rng.choice(["circle", "starfish", "ellipse"]),
                "panels": _log_int(rng, 128, 896) if fmm else _log_int(rng, 16, 256),
                "grid": _log_int(rng, 128, 768) if fmm else _log_int(rng, 16, 512), "alpha": _log(rng, 1.0, 1000.0),
                "layers": rng.choice(["both", "slp", "dlp"]),
                "precision": "fp64" if fmm else rng.choice(["fp64", "fp64", "mixed"]), "fmm": 40 if fmm else 0}
    if kind == "dirichlet":
        return {"kind": kind, "curve": rng.choice(["circle", "starfish", "ellipse"]), "panels": _log_int(rng, 32, 256),
                "grid": _log_int(rng, 16, 256), "alpha": _log(rng, 1.0, 500.0),
                "precision": rng.choice(["fp64", "mixed"])}
    if kind in ("grad", "stokes"):
        return {"kind": kind, "curve": rng.choice(["circle", "starfish", "ellipse"]), "panels": _log_int(rng, 32, 256),
                "grid": _log_int(rng, 16, 512 if kind == "grad" else 256), "alpha": _log(rng, 1.0, 500.0)}
    if kind == "batch":
        lo = rng.randint(16, 64)
        return {"kind": kind, "geometries": rng.randint(2, 16), "panels_lo": lo, "panels_hi": rng.randint(lo + 16, 160),
                "mix": rng.randint(1, 4)}
    if kind == "volume":
        return {"kind": kind, "n": _log_int(rng, 32, 256), "alpha": _log(rng, 2.0, 100.0),
                "precision": rng.choice(["fp64", "mixed"])}
    if kind == "box":
        return {"kind": kind, "M": rng.choice([64, 128, 256, 512]), "points": _log_int(rng, 100, 4096),
                "alpha": _log(rng, 2.0, 500.0)}
    return {"kind": "train", "batch": rng.randint(8, 128), "n_in": _log_int(rng, 256, 4096),
            "width": rng.randint(64, 256), "n_out": _log_int(rng, 64, 1024)}


# ---------------------------------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------------------------------
def _rng(case, seed):
    return np.random.default_rng([int(seed) & 0x7FFFFFFF, sum(case["kind"].encode())])


def _dev(a):
    return torch.as_tensor(np.ascontiguousarray(a), dtype=torch.float64, device=DEV)


def _shape(case):
    """The case's curve as plain numbers (kind, size, second axis, amplitude, arms)."""
    return {"circle": ("circle", 1.0, 1.0, 0.0, 0), "ellipse": ("ellipse", 1.3, 0.8, 0.0, 0),
            "starfish": ("starfish", 1.0, 1.0, 0.3, 5)}[case["curve"]]


def _discretize(shape, panels):
    kind, a, b, amp, arms = shape
    if kind == "ellipse":
        return wl.discretize(wl.Curve("ellipse", a=a, b=b), panels)
    if kind == "circle":
        return wl.discretize(wl.Curve("circle", R=a), panels)
    return wl.discretize(wl.Curve("starfish", R=a, A=amp, k=arms), panels)


def _grid(shape, n):
    """Points of an n x n grid inside the curve."""
    kind, a, b, amp, arms = shape
    g = np.linspace(-1.4, 1.4, n)
    x, y = (v.ravel() for v in np.meshgrid(g, g))
    th = np.arctan2(y, x)
    if kind == "ellipse":
        rho = 1.0 / np.hypot(np.cos(th) / a, np.sin(th) / b)
    else:
        rho = a * (1.0 + amp * np.cos(arms * th))
    keep = np.hypot(x, y) < (1.0 - MARGIN) * rho
    return x[keep], y[keep]


def _coeffs(rng):
    return rng.standard_normal(MODES) + 1j * rng.standard_normal(MODES)


def _fourier(c, theta):
    n = np.arange(MODES)
    return np.real(np.exp(1j * np.outer(theta, n)) @ c)


def _sources(rng):
    """Eight exterior point sources on the circle of radius 2."""
    return 2.0 * np.exp(1j * rng.uniform(0.0, TWO_PI, 8)), rng.standard_normal(8)


def _source_sum(x, y, alpha, zs, cs, shift):
    """sum c K0(alpha |x - z|) e^{alpha shift}; torch float64 tensors in and out."""
    v = torch.zeros_like(x)
    for z, c in zip(zs, cs):
        d = torch.hypot(x - z.real, y - z.imag)
        v += c * torch.special.scaled_modified_bessel_k0(alpha * d) * torch.exp(-alpha * (d - shift))
    return v


def _forces(rng):
    """Two exterior point forces on the circle of radius 2.2."""
    return 2.2 * np.exp(1j * rng.uniform(0.0, TWO_PI, 2)), rng.standard_normal((2, 2))


def _stokeslets(x, y, alpha, places, forces):
    """Velocity [2][n] of exterior modified stokeslets."""
    u = torch.zeros(2, x.numel(), dtype=torch.float64, device=x.device)
    for x0, (f1, f2) in zip(places, forces):
        rx, ry = x - x0.real, y - x0.imag
        z = alpha * torch.hypot(rx, ry)
        k0, k1 = torch.special.modified_bessel_k0(z), torch.special.modified_bessel_k1(z)
        s1 = (z * z * k0 + z * k1 - 1.0) / (TWO_PI * z * z)
        s2 = -(z * z * k0 + 2.0 * z * k1 - 2.0) / (TWO_PI * z ** 4)
        rf = rx * f1 + ry * f2
        u[0] += s1 * f1 + alpha * alpha * s2 * rx * rf
        u[1] += s1 * f2 + alpha * alpha * s2 * ry * rf
    return u


def _box_forcing(case, rng):
    """Sixteen Gaussian bumps per component inside the box, on the M x M grid (rows y)."""
    M, lb = case["M"], 4.0
    g = torch.arange(M, dtype=torch.float64, device=DEV) * (lb / M) - 0.5 * lb
    f = torch.zeros(2, M, M, dtype=torch.float64, device=DEV)
    for i in range(2):
        c, s, a = rng.uniform(-1.0, 1.0, (16, 2)), rng.uniform(0.08, 0.14, 16), rng.standard_normal(16)
        for k in range(16):
            gx = torch.exp(-((g - c[k, 0]) ** 2) / (2.0 * s[k] ** 2))
            gy = torch.exp(-((g - c[k, 1]) ** 2) / (2.0 * s[k] ** 2))
            f[i] += a[k] * gy[:, None] * gx[None, :]
    ang = rng.uniform(0.0, TWO_PI, case["points"])
    return f, 1.2 * np.cos(ang), 1.2 * np.sin(ang)


def _volume_points(case, rng):
    n = case["n"]
    g = np.linspace(-1.5, 1.5, n)
    h = float(g[1] - g[0])
    w1 = np.full(n, h)
    w1[0] = w1[-1] = 0.5 * h
    x, y = (v.ravel() for v in np.meshgrid(g, g))
    f = np.zeros(n * n)
    c, s, a = rng.uniform(-1.5, 1.5, (16, 2)), rng.uniform(0.05, 0.3, 16), rng.standard_normal(16)
    for b in range(16):
        f += a[b] * np.exp(-((x - c[b, 0]) ** 2 + (y - c[b, 1]) ** 2) / (2.0 * s[b] ** 2))
    return x, y, np.outer(w1, w1).ravel(), f, h


def _train_inputs(case, seed):
    """Smooth rows, features falling with the index as the differences of coefficients do."""
    gen = torch.Generator(device="cpu").manual_seed(int(seed) & 0x7FFFFFFF)
    B = case["batch"]
    X = torch.randn(B, case["n_in"], generator=gen)
    T = 0.5 * torch.randn(B, case["n_out"], generator=gen)
    sizes = [case["n_in"], case["width"], case["width"], case["n_out"]]
    p = []
    for a, b in zip(sizes[:-1], sizes[1:]):
        p += [(torch.rand(b * a, generator=gen) * 2.0 - 1.0) / math.sqrt(a), 0.01 * torch.randn(b, generator=gen)]
    return X, T, torch.cat(p), sizes


# ---------------------------------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------------------------------
def prepare(case, seed):
    rng = _rng(case, seed)
    kind = case["kind"]
    s = {"case": case}
    if kind == "volume":
        x, y, w, f, h = _volume_points(case, rng)
        s.update(x=_dev(x), y=_dev(y), w=_dev(w), f=_dev(f), h=h)
        return s
    if kind == "box":
        f, px, py = _box_forcing(case, rng)
        s.update(F=f, px=_dev(px), py=_dev(py), box=mhlp.Box(case["M"], -2.0, -2.0, 4.0, case["alpha"]))
        return s
    if kind == "train":
        X, T, p, sizes = _train_inputs(case, seed)
        net = mhlp.MLP(sizes[0], sizes[1], sizes[3], seed=0)
        net.set_params(p.to(DEV))
        s.update(net=net, X=X.to(DEV), T=T.to(DEV), p0=p.to(DEV))
        return s
    if kind == "batch":
        plans, rhs = [], []
        for i in range(case["geometries"]):
            if i % 2 == 0:
                a, b = rng.uniform(0.5, 1.5, 2)
                c = wl.Curve("ellipse", a=float(a), b=float(b))
            else:
                c = wl.Curve("starfish", R=1.0, A=float(rng.uniform(0.1, 0.3)), k=int(rng.integers(3, 8)))
            # panel counts and alphas spread over the range the same way for every seed
            u = (i * 0.6180339887 + 0.17 * case["mix"]) % 1.0
            v = (i * 0.7548776662 + 0.29 * case["mix"]) % 1.0
            g = wl.discretize(c, int(round(case["panels_lo"] + u * (case["panels_hi"] - case["panels_lo"]))))
            plans.append(mhlp.Plan(mhlp.Geometry(_dev(g.node_soa())), 10.0 ** (3.0 * v)))
            rhs += [_dev(_fourier(_coeffs(rng), g.theta)) for _ in range(4)]
        batch = mhlp.Batch(plans, 4)
        s.update(batch=batch, g=batch.pack(rhs))
        return s
    shape = _shape(case)
    g = _discretize(shape, case["panels"])
    tx, ty = (_dev(v) for v in _grid(shape, case["grid"]))
    alpha = case["alpha"]
    geom = mhlp.Geometry(_dev(g.node_soa()))
    s.update(geom=geom, off=mhlp.Plan(geom, alpha, tx, ty, stokes=kind == "stokes"))
    if kind in ("eval", "grad"):
        s.update(sigma=_dev(_fourier(_coeffs(rng), g.theta)), mu=_dev(_fourier(_coeffs(rng), g.theta)))
        if case.get("fmm"):
            s["off"].set_fmm(case["fmm"])
        return s
    x, y = _dev(g.x), _dev(g.y)
    s["on"] = mhlp.Plan(geom, alpha, stokes=kind == "stokes")
    if kind == "dirichlet":
        zs, cs = _sources(rng)
        s["g"] = _source_sum(x, y, alpha, zs, cs, _shift(x, y, zs))
    else:
        s["g"] = _stokeslets(x, y, alpha, *_forces(rng))
    return s


def _shift(x, y, zs):
    return min(float(torch.hypot(x - z.real, y - z.imag).min()) for z in zs)


PRECISION = {"fp64": mhlp.FP64, "mixed": mhlp.MIXED}


def run(state):
    case = state["case"]
    kind = case["kind"]
    if kind == "eval":
        p = PRECISION[case["precision"]]
        if case["layers"] == "slp":
            return mhlp.eval_slp(state["off"], state["sigma"], precision=p)
        if case["layers"] == "dlp":
            return mhlp.eval_dlp(state["off"], state["mu"], precision=p)
        return list(mhlp.eval_layer(state["off"], sigma=state["sigma"], mu=state["mu"], precision=p))
    if kind == "dirichlet":
        mu, _ = mhlp.gmres_solve(state["on"], state["g"], tol=1e-10, restart=200,
                                 precision=PRECISION[case["precision"]])
        return {"mu": mu, "u": mhlp.eval_dlp(state["off"], mu)}
    if kind == "grad":
        return list(mhlp.eval_grad(state["off"], sigma=state["sigma"], mu=state["mu"]))
    if kind == "stokes":
        mu, _ = mhlp.stokes_gmres_solve(state["on"], state["g"], tol=1e-10, restart=200)
        return {"mu": mu, "u": mhlp.stokes_eval(state["off"], mu), "grad": mhlp.stokes_eval_grad(state["off"], mu)}
    if kind == "batch":
        mu, _ = state["batch"].gmres(state["g"], tol=1e-10)
        return mu
    if kind == "volume":
        return mhlp.volume_eval(state["x"], state["y"], state["w"], state["f"], case["alpha"], state["h"],
                                precision=PRECISION[case["precision"]])[0]
    if kind == "box":
        return list(state["box"].particular(state["F"], want_u=True, want_grad=True, px=state["px"], py=state["py"]))
    # train: the same step from the same weights in every pass
    net = state["net"]
    net.set_params(state["p0"])
    loss, grad = net.loss_grad(state["X"], state["T"])
    net.adam_step(lr=1e-3)
    return {"loss": loss, "grad": grad, "params": net.get_params()}


# ---------------------------------------------------------------------------------------------------
# what a pass cannot do without: each input read once, each output written once; the operations of the
# contractions that have no shorter form (network, transforms), none where a fast summation has O(N + M)
# ---------------------------------------------------------------------------------------------------
def _inside(case):
    area = {"circle": math.pi, "ellipse": math.pi * 1.04, "starfish": math.pi * 1.045}[case["curve"]]
    return area * ((case["grid"] - 1) / 2.8) ** 2


def work(case):
    kind = case["kind"]
    if kind == "train":
        B, sizes = case["batch"], [case["n_in"], case["width"], case["width"], case["n_out"]]
        w = sum(a * b for a, b in zip(sizes[:-1], sizes[1:]))
        # weights read from the start copy, moments, gradient and the two results; three products per layer
        return {"bytes": 4.0 * (9 * w + B * (sizes[0] + sizes[3])), "flops": 6.0 * B * w - 2.0 * B * sizes[0] * sizes[1]}
    if kind == "volume":
        return {"bytes": 8.0 * 5 * case["n"] ** 2, "flops": 0.0}
    if kind == "box":
        m2 = case["M"] ** 2
        return {"bytes": 8.0 * (8 * m2 + 4 * case["points"]), "flops": 8 * 2.5 * m2 * math.log2(m2)}
    if kind == "batch":
        n = 16 * case["geometries"] * 0.5 * (case["panels_lo"] + case["panels_hi"])
        return {"bytes": 8.0 * n * (9 + 2 * 4), "flops": 0.0}
    n, m = 16.0 * case["panels"], _inside(case)
    out = {"eval": 2 if case.get("layers") == "both" else 1, "dirichlet": 1, "grad": 4, "stokes": 6}[kind]
    dens = {"eval": out, "dirichlet": 2, "grad": 2, "stokes": 4}[kind]
    return {"bytes": 8.0 * (n * (9 + dens) + m * (2 + out)), "flops": 0.0}


# ---------------------------------------------------------------------------------------------------
# 64-bit references
# ---------------------------------------------------------------------------------------------------
def _curve_points(shape, th):
    """x, y, dx, dy of the curve at the parameters th (the discretisation's parametrisation)."""
    kind, a, b, amp, arms = shape
    c, s = torch.cos(th), torch.sin(th)
    if kind == "ellipse":
        return a * c, b * s, -a * s, b * c
    r = a * (1.0 + amp * torch.cos(arms * th))
    dr = -a * amp * arms * torch.sin(arms * th)
    return r * c, r * s, dr * c - r * s, dr * s + r * c


def _series(c, th):
    v = torch.zeros_like(th)
    for n, z in enumerate(c):
        v += z.real * torch.cos(n * th) - z.imag * torch.sin(n * th)
    return v


def _layers_exact(shape, alpha, cs, cd, tx, ty, grad):
    """S[sigma], D[mu] (grad: their gradients) by the periodic trapezoid rule in the curve's parameter, as
    many points as the target's distance asks for: its error falls as exp(-points * distance / speed)."""
    dev = tx.device
    coarse = torch.arange(8192, dtype=torch.float64, device=dev) * (TWO_PI / 8192)
    qx, qy, _, _ = _curve_points(shape, coarse)
    dist = torch.empty_like(tx)
    for i in range(0, tx.numel(), 8192):
        sl = slice(i, i + 8192)
        dist[sl] = torch.sqrt(((tx[sl, None] - qx) ** 2 + (ty[sl, None] - qy) ** 2).min(dim=1).values)
    # the nearest of 8192 points is further than the curve by at most the square of half their spacing
    dist = torch.sqrt(torch.clamp(dist ** 2 - (0.5 * 1.9 * TWO_PI / 8192) ** 2, min=(0.25 * MARGIN) ** 2))
    out = torch.zeros(4 if grad else 2, tx.numel(), dtype=torch.float64, device=dev)
    level = torch.clamp(torch.floor(torch.log2(0.5 / dist)), min=0)
    for lv in torch.unique(level).tolist():
        sel = torch.nonzero(level == lv).ravel()
        n = int(352 * 2 ** lv)
        th = torch.arange(n, dtype=torch.float64, device=dev) * (TWO_PI / n)
        for a in range(0, n, 16384):
            t = th[a:a + 16384]
            x, y, dx, dy = _curve_points(shape, t)
            q = _series(cs, t) * torch.hypot(dx, dy) / n
            mx, my = -dy * _series(cd, t) / n, dx * _series(cd, t) / n  # inward normal times speed
            step = max(1, 4_000_000 // t.numel())
            for b in range(0, sel.numel(), step):
                k = sel[b:b + step]
                ex, ey = tx[k, None] - x, ty[k, None] - y
                r2 = ex * ex + ey * ey
                z = alpha * torch.sqrt(r2)
                k0, k1 = torch.special.modified_bessel_k0(z), torch.special.modified_bessel_k1(z)
                A = alpha * k1 / torch.sqrt(r2)
                dot = ex * mx + ey * my
                if grad:
                    B = dot * (alpha * alpha * k0 + 2.0 * A) / r2
                    out[0, k] -= (A * ex) @ q
                    out[1, k] -= (A * ey) @ q
                    out[2, k] += (A * mx - B * ex).sum(dim=1)
                    out[3, k] += (A * my - B * ey).sum(dim=1)
                else:
                    out[0, k] += k0 @ q
                    out[1, k] += (A * dot).sum(dim=1)
    return out


def _box_exact(case, rng):
    F, px, py = _box_forcing(case, rng)
    M, lb, a2 = case["M"], 4.0, case["alpha"] ** 2
    k1 = torch.fft.fftfreq(M, 1.0 / M, device=DEV).to(torch.float64)
    keep = (k1 != -M // 2).to(torch.float64)
    k = k1 * (TWO_PI / lb)
    kx, ky, ok = k[None, :], k[:, None], keep[None, :] * keep[:, None]
    k2 = kx * kx + ky * ky
    fh = torch.fft.fft2(F) * ok / (M * M)
    kf = (kx * fh[0] + ky * fh[1]) / torch.where(k2 == 0, torch.ones_like(k2), k2)
    uh = torch.stack([fh[0] - kx * kf, fh[1] - ky * kf]) / (a2 + k2)
    back = lambda v: torch.fft.ifft2(v).real * (M * M)  # noqa: E731
    grad = torch.stack([back(1j * q * uh[i]) for i in range(2) for q in (kx, ky)])
    ex = torch.exp(1j * torch.outer(_dev(px) + 2.0, k))
    ey = torch.exp(1j * torch.outer(_dev(py) + 2.0, k))
    up = torch.stack([((ex @ uh[i].T.contiguous()) * ey).sum(dim=1).real for i in range(2)])
    return [back(uh), grad, up]


def _volume_exact(case, rng):
    x, y, w, f, h = _volume_points(case, rng)
    x, y, q, alpha = _dev(x), _dev(y), _dev(w * f), case["alpha"]
    n = x.numel()
    u = torch.empty_like(x)
    for i in range(0, n, 1024):
        z = alpha * torch.hypot(x[i:i + 1024, None] - x, y[i:i + 1024, None] - y)
        k0 = torch.special.modified_bessel_k0(z)
        u[i:i + 1024] = torch.where(z == 0, torch.zeros_like(z), k0) @ q / TWO_PI
    t, lam = np.polynomial.legendre.leggauss(200)
    th = 0.125 * math.pi * (t + 1.0)
    z = alpha * torch.as_tensor(h / (2.0 * np.cos(th)))
    cell = float((torch.as_tensor(lam) * (1.0 - z * torch.special.modified_bessel_k1(z))).sum()) * 0.125 * math.pi
    return u + q * (8.0 * cell / (alpha * alpha) / TWO_PI) / (h * h)


def _train_exact(case, seed):
    X, T, p, sizes = _train_inputs(case, seed)
    X, T, p = (v.to(DEV, torch.float64) for v in (X, T, p))
    p.requires_grad_(True)
    h, at = X, 0
    for layer, (a, b) in enumerate(zip(sizes[:-1], sizes[1:])):
        W, c = p[at:at + a * b].view(b, a), p[at + a * b:at + a * b + b]
        at += a * b + b
        h = h @ W.T + c
        if layer < 2:
            h = torch.nn.functional.gelu(h, approximate="tanh")
    loss = ((h - T) ** 2).mean()
    (grad,) = torch.autograd.grad(loss, p)
    # the first Adam step moves every parameter by lr * g / (|g| + eps)
    return {"loss": loss.detach().reshape(1), "grad": grad, "params": p.detach() - 1e-3 * grad / (grad.abs() + 1e-8)}


def exact(case, seed):
    rng = _rng(case, seed)
    kind = case["kind"]
    if kind == "train":
        return _train_exact(case, seed)
    if kind == "volume":
        return _volume_exact(case, rng)
    if kind == "box":
        return _box_exact(case, rng)
    if kind == "batch":
        return None  # densities of dense systems without a closed form
    shape, alpha = _shape(case), case["alpha"]
    tx, ty = (_dev(v) for v in _grid(shape, case["grid"]))
    if kind in ("eval", "grad"):
        cs, cd = _coeffs(rng), _coeffs(rng)
        v = _layers_exact(shape, alpha, cs, cd, tx, ty, kind == "grad")
        if kind == "grad":
            return [v[:2], v[2:]]
        return {"both": [v[0], v[1]], "slp": v[0], "dlp": v[1]}[case["layers"]]
    if kind == "dirichlet":
        zs, cs = _sources(rng)
        g = _discretize(shape, case["panels"])
        return {"mu": None, "u": _source_sum(tx, ty, alpha, zs, cs, _shift(_dev(g.x), _dev(g.y), zs))}
    return {"mu": None, "u": _stokeslets(tx, ty, alpha, *_forces(rng)), "grad": None}
