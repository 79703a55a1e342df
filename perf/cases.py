"""Workloads of the solver as a user's program runs them, through the package's public calls.

``listed()`` names the standing ones, ``draw(rng)`` gives others of the same ranges, ``prepare`` makes what such a
program holds before the call (inputs, workspaces, and the plan or factor it keeps), ``run`` makes one pass,
``work`` counts what the pass cannot do without and ``exact`` computes its result with plain torch in 64 bits where
that is quick.

Grids are n x n with n = leaf * 2^m on the unit square and about 10 to 20 nodes per wavelength.  The kinds:

  setup      lsh_build + lsh_solve: one problem from scratch (plan, factor, solve)
  solve      lsh_solve with a kept factor: new incident fields on a known scatterer
  gradient   receiver_field forward and backward with a kept plan: one step of an inversion
  batch      lsh_batch_factor on kept plans, then each instance's solve: many uneven problems with new potentials
  operator   lsh_apply_operator: the FFT matvec, as a caller's own iteration uses it
  receivers  lsh_eval_points and its adjoint: fields at off-grid points and their back-propagation
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_12718_amd import lsh

MAXIT = 100


def listed():
    return [
        # the smallest whole solve (the smoke run's grid), at direct-solver accuracy: host time, launches and latency
        {"name": "setup-32-fine", "kind": "setup", "n": 32, "leaf": 8, "waves": 4.0, "order": 4, "hbs_order": 4,
         "tol": 1e-10, "width": 3, "prec": "fp64", "full": 0, "nrhs": 1, "field": "gauss", "gmres": 1e-10},
        # the direct-solver mode: the 10th-order matrix itself compressed to 1e-10, FGMRES as the final polish
        {"name": "setup-64-direct", "kind": "setup", "n": 64, "leaf": 8, "waves": 5.0, "order": 10,
         "hbs_order": 10, "tol": 1e-10, "width": 3, "prec": "fp64", "full": 0, "nrhs": 1, "field": "bumps",
         "gmres": 1e-12},
        # an ordinary single problem: bumps on 256 x 256, 20 wavelengths
        {"name": "setup-256", "kind": "setup", "n": 256, "leaf": 8, "waves": 20.0, "order": 6, "hbs_order": 4,
         "tol": 1e-4, "width": 2, "prec": "fp32", "full": 0, "nrhs": 1, "field": "bumps", "gmres": 1e-10},
        # a side that is not a power of two (leaf 6), double-precision factor, several incident fields
        {"name": "setup-384-fp64", "kind": "setup", "n": 384, "leaf": 6, "waves": 37.5, "order": 8, "hbs_order": 4,
         "tol": 1e-4, "width": 2, "prec": "fp64", "full": 0, "nrhs": 3, "field": "bumps", "gmres": 1e-10},
        # the largest: 1024 x 1024, 100 wavelengths, as the benchmark builds it
        {"name": "setup-1024", "kind": "setup", "n": 1024, "leaf": 8, "waves": 100.0, "order": 10, "hbs_order": 4,
         "tol": 1e-4, "width": 2, "prec": "fp32", "full": 1, "nrhs": 1, "field": "fourier", "gmres": 1e-10},
        # the same scatterer lit from another angle: the factor is kept
        {"name": "solve-1024", "kind": "solve", "n": 1024, "leaf": 8, "waves": 100.0, "order": 10, "hbs_order": 4,
         "tol": 1e-4, "width": 2, "prec": "fp32", "full": 1, "nrhs": 1, "field": "fourier", "gmres": 1e-10},
        # eight plane waves on one scatterer at once
        {"name": "solve-512x8", "kind": "solve", "n": 512, "leaf": 8, "waves": 40.0, "order": 10, "hbs_order": 4,
         "tol": 1e-4, "width": 2, "prec": "fp32", "full": 0, "nrhs": 8, "field": "bumps", "gmres": 1e-10},
        # one inversion step: factor, 8 forward solves, 64 receivers, 8 adjoint solves, gradient in b
        {"name": "gradient-512x8", "kind": "gradient", "n": 512, "leaf": 8, "waves": 40.0, "order": 10,
         "hbs_order": 4, "tol": 1e-4, "width": 2, "prec": "fp32", "full": 0, "nrhs": 8, "npts": 64,
         "field": "bumps", "gmres": 1e-10},
        # many small uneven problems (sides 64 to 256) with new potentials on kept plans
        {"name": "batch-16", "kind": "batch", "count": 16, "mix": 3000, "order": 6, "hbs_order": 4, "tol": 1e-4,
         "width": 2, "prec": "fp32", "full": 0, "nrhs": 1, "field": "bumps", "gmres": 1e-10},
        # one matvec on a small grid: a few microseconds of work
        {"name": "operator-64", "kind": "operator", "n": 64, "leaf": 8, "waves": 6.4, "order": 4, "nrhs": 1,
         "field": "gauss"},
        # several vectors on a grid whose doubled side is far below its padded length
        {"name": "operator-640x4", "kind": "operator", "n": 640, "leaf": 5, "waves": 60.0, "order": 10, "nrhs": 4,
         "field": "fourier"},
        # eight fields at 64 receivers, and the receivers' residuals back on the grid
        {"name": "receivers-512x8", "kind": "receivers", "n": 512, "leaf": 8, "waves": 40.0, "order": 4, "nrhs": 8,
         "npts": 64},
    ]


def draw(rng):
    kind = rng.choice(["setup", "setup", "setup", "solve", "solve", "gradient", "batch", "operator", "receivers"])
    c = {"kind": kind, "hbs_order": 4, "tol": 1e-4, "width": 2, "prec": rng.choice(["fp32", "fp32", "fp64"]),
         "full": rng.choice([0, 0, 1]), "nrhs": 1, "field": rng.choice(["bumps", "fourier"]), "gmres": 1e-10,
         "order": rng.choice([4, 6, 8, 10])}
    if kind == "batch":
        c |= {"count": rng.randint(3, 20), "mix": rng.randrange(1 << 20), "full": 0}
        return c

    def side(lo, hi):
        """(n, leaf): n = leaf * 2^m in [lo, hi], leaf 5 to 8, about even over the logarithm."""
        want = lo * (hi / lo) ** rng.random()
        leaf = rng.choice([5, 6, 7, 8])
        m = max(1, round(math.log2(want / leaf)))
        while leaf << m > hi:
            m -= 1
        while leaf << m < lo:
            m += 1
        return leaf << m, leaf

    if kind == "setup" and rng.random() < 0.3:  # direct-solver accuracy, small grids
        order = rng.choice([4, 6, 10])
        n, leaf = side(32, 64)
        c |= {"n": n, "leaf": leaf, "order": order, "hbs_order": order, "tol": rng.choice([1e-8, 1e-9, 1e-10]),
              "width": 3, "prec": "fp64", "full": 0, "gmres": 1e-12}
    else:
        lo, hi = {"setup": (64, 640), "solve": (64, 640), "gradient": (64, 448), "operator": (40, 1024),
                  "receivers": (64, 640)}[kind]
        n, leaf = side(lo, hi)
        c |= {"n": n, "leaf": leaf}
        most = {"setup": 4, "solve": 8, "gradient": 8, "operator": 8, "receivers": 8}[kind]
        c["nrhs"] = rng.randint(1, most)
    if kind in ("gradient", "receivers"):
        c["npts"] = int(16 * 16 ** rng.random()) if kind == "gradient" else int(16 * 16 ** rng.random()) | 1
    c["waves"] = round(n / 10 * rng.uniform(0.5, 1.0), 3)
    return c


# ---- inputs ----

def _gen(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(int(seed))
    return g


def _uniform(g, shape, lo, hi):
    return lo + (hi - lo) * torch.rand(shape, generator=g, device="cuda", dtype=torch.float64)


def _nodes(n):
    return -0.5 + (torch.arange(n, device="cuda", dtype=torch.float64) + 0.5) / n


def _potential(g, n, field):
    """A smooth scatterer on the unit square, below 1 where the medium is slower than the background."""
    t = _nodes(n)
    if field == "gauss":
        a, w = _uniform(g, (1,), 0.4, 0.6), _uniform(g, (1,), 0.12, 0.18)
        e = torch.exp(-t ** 2 / (2 * w ** 2))
        return a * e[:, None] * e[None, :]
    if field == "bumps":  # ten Gaussians of either sign, clipped below 1
        c, w, a = _uniform(g, (2, 10), -0.4, 0.4), _uniform(g, (10,), 0.03, 0.1), _uniform(g, (10,), -1.5, 0.9)
        e = torch.exp(-(t[None, :, None] - c[:, None, :]) ** 2 / (2 * w ** 2))
        return torch.clamp((e[1] * a) @ e[0].T, max=0.95).contiguous()
    # random Fourier modes of up to 20 cycles, and no more than 5 nodes to a cycle, scaled to [-1, 0.9]
    K = max(2, min(20, n // 12))
    k = torch.arange(-K, K + 1, device="cuda", dtype=torch.float64)
    coef = torch.randn((2, 2 * K + 1, 2 * K + 1), generator=g, device="cuda", dtype=torch.float64)
    coef = torch.complex(coef[0], coef[1]) * (k[:, None] ** 2 + k[None, :] ** 2 <= K * K)
    ph = torch.exp(2j * math.pi * t[:, None] * k[None, :])
    f = (ph @ coef @ ph.T).real
    return (-1 + 1.9 * (f - f.min()) / (f.max() - f.min())).contiguous()


def _plane_waves(g, n, kappa, nrhs):
    t = _nodes(n)
    th = 2 * math.pi * (torch.arange(nrhs, device="cuda", dtype=torch.float64) / nrhs + _uniform(g, (1,), 0, 1))
    ph = torch.cos(th)[:, None, None] * t[None, None, :] + torch.sin(th)[:, None, None] * t[None, :, None]
    return torch.exp(1j * kappa * ph)


def _receivers(g, npts):
    th = 2 * math.pi * (torch.arange(npts, device="cuda", dtype=torch.float64) / npts + _uniform(g, (1,), 0, 1))
    return torch.stack([0.75 * torch.cos(th), 0.75 * torch.sin(th)], dim=1).contiguous()


def _complex_normal(g, shape):
    x = torch.randn((2,) + tuple(shape), generator=g, device="cuda", dtype=torch.float64)
    return torch.complex(x[0], x[1])


def _instances(case):
    """(n, leaf, wavelengths) of a batch: sides 64 to 256, 5 wavelengths to 10 nodes each (at most 20)."""
    rng = np.random.default_rng(case["mix"])
    out = []
    for _ in range(case["count"]):
        n = int(rng.choice([64, 96, 128, 192, 256]))
        out.append((n, 8 if n in (64, 128, 256) else 6, float(rng.uniform(5, min(20, n / 10)))))
    return out


def _inputs(case, seed):
    """The arrays of one case; the same for the same seed."""
    g = _gen(seed)
    kind = case["kind"]
    if kind == "batch":
        return [{"b": _potential(g, n, case["field"]), "u": _plane_waves(g, n, 2 * math.pi * waves, 1)}
                for n, _, waves in _instances(case)]
    n, nrhs, kappa = case["n"], case["nrhs"], 2 * math.pi * case["waves"]
    if kind == "operator":
        return {"b": _potential(g, n, case["field"]), "x": _complex_normal(g, (nrhs, n, n))}
    if kind == "receivers":
        return {"sigma": _complex_normal(g, (nrhs, n, n)), "xy": _receivers(g, case["npts"]),
                "g": _complex_normal(g, (nrhs, case["npts"]))}
    s = {"b": _potential(g, n, case["field"]), "u": _plane_waves(g, n, kappa, nrhs)}
    if kind == "gradient":
        s["xy"] = _receivers(g, case["npts"])
        s["data"] = 0.1 * _complex_normal(g, (nrhs, case["npts"]))
    return s


def _options(case):
    return {"op_order": case["order"], "leaf": case["leaf"], "tol": case["tol"], "proxy_width": case["width"],
            "prec": case["prec"], "hbs_order": case["hbs_order"], "full_levels": case["full"]}


def prepare(case, seed):
    kind = case["kind"]
    s = {"case": case, "in": _inputs(case, seed)}
    if kind == "batch":
        s["plans"] = [lsh.Plan(n, 2 * math.pi * waves, op_order=case["order"], leaf=leaf, tol=case["tol"],
                               proxy_width=case["width"], prec=case["prec"]) for n, leaf, waves in _instances(case)]
        return s
    n, kappa = case["n"], 2 * math.pi * case["waves"]
    s["kappa"] = kappa
    if kind == "setup":  # the build's workspaces, reused from problem to problem
        s["ws"] = lsh.build_workspaces(n, kappa, **_options(case))
    elif kind == "solve":
        s["plan"] = lsh.Plan(n, kappa, **_options(case))
        s["factor"] = lsh.Factor(s["plan"], s["in"]["b"])
    elif kind == "gradient":
        s["plan"] = lsh.Plan(n, kappa, **_options(case))
    else:  # the FFT operator and the receivers need no compressed levels: a coarse plan serves them
        s["plan"] = lsh.Plan(n, kappa, op_order=case["order"], leaf=case["leaf"], tol=1e-2, proxy_width=1)
    return s


# ---- one pass ----

def run(s):
    case, x = s["case"], s["in"]
    kind = case["kind"]
    if kind == "setup":
        P, F = lsh.build(case["n"], s["kappa"], x["b"], workspaces=s["ws"], **_options(case))
        sigma, u, _, _ = F.solve(x["u"], tol=case["gmres"], maxit=MAXIT)
        F.close()
        P.close()
        return {"sigma": sigma, "u": u}
    if kind == "solve":
        sigma, u, _, _ = s["factor"].solve(x["u"], tol=case["gmres"], maxit=MAXIT)
        return {"sigma": sigma, "u": u}
    if kind == "gradient":
        b = x["b"].detach().requires_grad_(True)
        ur = lsh.receiver_field(b, x["u"], x["xy"], s["plan"], tol=case["gmres"], maxit=MAXIT)
        misfit = 0.5 * (ur - x["data"]).abs().square().sum()
        misfit.backward()
        return {"field": ur.detach(), "grad": b.grad}
    if kind == "batch":
        factors = lsh.batch_factor(s["plans"], [v["b"] for v in x])
        out = []
        for F, v in zip(factors, x):
            sigma, u, _, _ = F.solve(v["u"], tol=case["gmres"], maxit=MAXIT)
            out.append({"sigma": sigma, "u": u})
            F.close()
        return out
    if kind == "operator":
        return s["plan"].apply_operator(x["b"], x["x"])
    return {"field": s["plan"].eval_points(x["sigma"], x["xy"]),
            "back": s["plan"].eval_points_adjoint(x["g"], x["xy"])}


# ---- what a pass cannot do without ----

def _tree(n, leaf):
    """(boxes, skeleton size) per level below the root, leaves last: a box keeps about its perimeter's nodes."""
    out, sx, sy, boxes = [], n, n, 1
    while sx > leaf or sy > leaf:
        sx, sy = (sx // 2, sy) if sx == sy else (sx, sy // 2)
        boxes *= 2
        out.append((boxes, min(sx * sy, 2 * (sx + sy) - 4)))
    return out


def _plan_flops(n, leaf):
    """Row IDs: per level, k pivots of the 2k' candidate rows against as many proxy columns (the Gram and its
    factorisation, complex); one per level by translation invariance."""
    lv = _tree(n, leaf) + [(0, leaf * leaf // 2)]
    return sum(8 * (2 * lv[i + 1][1]) ** 2 * (lv[i][1] + lv[i + 1][1]) for i in range(len(lv) - 1))


def _factor_flops(n, leaf):
    """Leaf inverses, and per parent box the Woodbury merge (rank about c / 3) and the scattering matrix."""
    lv, f = _tree(n, leaf), 8 * (n * n // leaf ** 2) * leaf ** 6
    parents = [(1, 0)] + lv[:-1]
    for (boxes, k), (_, c) in zip(parents, lv):
        r = c // 3
        f += boxes * 8 * (2 * c * c * r + 4 * c * r * r + 8 * r ** 3 + (2 * c) * k * (2 * c - k))
    return f


def _factor_values(n, leaf):
    """Entries that one application of the inverse reads: leaf inverses twice, merge factors, scattering matrices."""
    lv, v = _tree(n, leaf), 2 * n * n * leaf * leaf
    for (boxes, c) in lv:
        r = c // 3
        v += boxes // 2 * (2 * c * c + 2 * (4 * r * r + 2 * c * r))
    return v


def _solve_work(case, n, leaf, nrhs):
    """About 5 iterations: the factor read once each, the basis and the FFT's vectors, the operator's transform."""
    iters = 2 if case["tol"] < 1e-7 else 5
    e = 8 if case["prec"] == "fp32" else 16
    m = 2 * n
    byts = iters * (e * _factor_values(n, leaf) + nrhs * 16 * n * n * (6 + iters)) + 48 * n * n * nrhs
    flops = iters * nrhs * (8 * _factor_values(n, leaf) + 10 * m * m * math.log2(m * m))
    return byts, flops


def work(case):
    kind = case["kind"]
    if kind == "batch":
        byts = flops = 0
        for n, leaf, _ in _instances(case):
            sb, sf = _solve_work(case, n, leaf, 1)
            byts, flops = byts + sb, flops + sf + _factor_flops(n, leaf)
        return {"bytes": byts, "flops": flops}
    n, nrhs = case["n"], case["nrhs"]
    if kind == "operator":
        m = 2 * n
        return {"bytes": 16 * 2 * n * n * nrhs + 8 * n * n + 16 * (n + 1) ** 2,
                "flops": nrhs * (10 * m * m * math.log2(m * m) + 8 * m * m)}
    if kind == "receivers":  # each pair's kernel value once per direction, about 100 operations, and its products
        pairs = n * n * case["npts"]
        return {"bytes": 2 * 16 * n * n * nrhs + 32 * case["npts"] * nrhs, "flops": pairs * 2 * (100 + 8 * nrhs)}
    byts, flops = _solve_work(case, n, case["leaf"], nrhs)
    if kind == "setup":
        flops += _plan_flops(n, case["leaf"]) + _factor_flops(n, case["leaf"])
    elif kind == "gradient":
        byts, flops = 2 * byts, 2 * flops + _factor_flops(n, case["leaf"])
    return {"bytes": byts, "flops": flops}


# ---- the same results from plain torch in 64 bits ----

# Correction weights tau' on the orbits of (0,0), (1,0), (1,1), (2,0), (2,1), (3,0) under the square's symmetries,
# by order: solutions of the lattice-zeta moment equations of the punctured trapezoidal rule for ln r.
_ORBITS = [(0, 0), (1, 0), (1, 1), (2, 0), (2, 1), (3, 0)]
_TAU = {
    4: [-1.3105329259115095],
    6: [-1.2133459579012367, -0.02429674200256823],
    8: [-1.1882171416684366, -0.030413000735379225, -0.003390020017183395, 0.003224074691794445],
    10: [-1.1765194993167498, -0.03306670571137943, -0.006162677466595331, 0.005533252534429898,
         0.00034658218117649195, -0.0005003903674980727],
}


def _hankel(x):
    """H0(x) = (-2i / pi) e^(ix) times the integral of e^(-x s^2) / sqrt(s^2 - 2i) over the real line, by the
    trapezoidal rule (exponentially convergent; 1e-15 for x >= 0.1)."""
    step = torch.clamp(0.5 / torch.sqrt(x), max=0.15)
    smallest = float(x.min())
    acc = torch.zeros_like(x, dtype=torch.complex128)
    for i in range(int(math.sqrt(38 / smallest) / min(0.15, 0.5 / math.sqrt(smallest))) + 2):
        s2 = (i * step) ** 2
        term = torch.exp(-x * s2) / torch.sqrt(torch.complex(s2, torch.full_like(s2, -2.0)))
        acc += term if i else 0.5 * term
    return (-4j / math.pi) * step * acc * torch.exp(1j * x)


def _green(kr):
    """(i/4) H0(kr)."""
    return 0.25j * _hankel(kr)


class _Operator:
    """K by circulant embedding: K_ij = h^2 [(i/4) H0(kappa |x_i - x_j|) + tau]."""

    def __init__(self, n, kappa, order):
        h, m = 1.0 / n, 2 * n
        d = torch.arange(m, device="cuda", dtype=torch.float64)
        d = torch.minimum(d, m - d)
        r = torch.sqrt(d[:, None] ** 2 + d[None, :] ** 2)
        K = _green(kappa * h * r.clamp(min=1.0))
        c0 = 0.25j - (math.log(kappa * h / 2) + float(np.euler_gamma)) / (2 * math.pi)
        K[0, 0] = torch.tensor(c0, dtype=torch.complex128, device="cuda")
        for (p, q), w in zip(_ORBITS, _TAU[order]):
            kr = torch.tensor([kappa * h * math.hypot(p, q)], dtype=torch.float64, device="cuda")
            j0 = _hankel(kr)[0].real if p else 1.0
            t = torch.complex(torch.as_tensor(-w / (2 * math.pi) * j0, dtype=torch.float64, device="cuda"),
                              torch.zeros((), dtype=torch.float64, device="cuda"))
            for y, x in {(sy * v, sx * u) for u, v in ((p, q), (q, p)) for sx in (1, -1) for sy in (1, -1)}:
                K[y % m, x % m] += t
        self.n, self.khat = n, torch.fft.fft2(h * h * K)

    def __call__(self, x):
        m = 2 * self.n
        return torch.fft.ifft2(self.khat * torch.fft.fft2(x, s=(m, m)))[..., :self.n, :self.n]


def _gmres(apply, f, tol=1e-13, maxit=900):
    """Full GMRES (Gram-Schmidt twice); None where it has not converged."""
    shape, beta = f.shape, float(torch.linalg.vector_norm(f))
    V = torch.zeros((maxit + 1, f.numel()), dtype=f.dtype, device=f.device)
    V[0] = f.reshape(-1) / beta
    R, cs, g = np.zeros((maxit + 1, maxit), complex), [], np.zeros(maxit + 1, complex)
    g[0] = beta
    for j in range(maxit):
        w = apply(V[j].reshape(shape)).reshape(-1)
        c1 = torch.mv(V[:j + 1].conj(), w)
        w = w - torch.mv(V[:j + 1].T, c1)
        c2 = torch.mv(V[:j + 1].conj(), w)
        w = w - torch.mv(V[:j + 1].T, c2)
        norm = torch.linalg.vector_norm(w)
        V[j + 1] = w / norm
        h = np.append((c1 + c2).cpu().numpy(), float(norm))
        for i, (c, s) in enumerate(cs):
            h[i], h[i + 1] = c * h[i] + s * h[i + 1], -np.conj(s) * h[i] + c * h[i + 1]
        t = math.hypot(abs(h[j]), abs(h[j + 1]))
        c = abs(h[j]) / t
        s = (h[j] / abs(h[j]) if h[j] else 1.0) * np.conj(h[j + 1]) / t
        cs.append((c, s))
        h[j], h[j + 1] = c * h[j] + s * h[j + 1], 0.0
        R[:j + 2, j] = h
        g[j], g[j + 1] = c * g[j], -np.conj(s) * g[j]
        if abs(g[j + 1]) <= tol * beta:
            y = np.linalg.solve(R[:j + 1, :j + 1], g[:j + 1])
            return torch.mv(V[:j + 1].T, torch.from_numpy(y).to(f.device)).reshape(shape)
    return None


def _exact_solve(n, kappa, order, b, u):
    """sigma and K sigma per incident field; None where GMRES gives up."""
    K = _Operator(n, kappa, order)

    def A(x):
        return x + kappa ** 2 * b * K(x)

    out = []
    for v in u:
        f = -kappa ** 2 * b * v
        x = _gmres(A, f)
        if x is None:
            return None
        out.append(x)
    sigma = torch.stack(out)
    return {"sigma": sigma, "u": K(sigma)}


def _exact_points(n, kappa, xy):
    """The receivers' rows (npts, n*n): h^2 (i/4) H0(kappa |x_r - x_j|)."""
    t = _nodes(n)
    out = []
    for p in xy:
        r = torch.sqrt((t[None, :] - p[0]) ** 2 + (t[:, None] - p[1]) ** 2)
        out.append(_green(kappa * r).reshape(-1) / (n * n))
    return torch.stack(out)


def exact(case, seed):
    x, kind = _inputs(case, seed), case["kind"]
    if kind == "batch":
        out = []
        for (n, _, waves), v in zip(_instances(case), x):
            e = _exact_solve(n, 2 * math.pi * waves, case["order"], v["b"], v["u"]) if n <= 96 else None
            out.append(e or {"sigma": None, "u": None})
        return out
    n, nrhs, kappa = case["n"], case["nrhs"], 2 * math.pi * case["waves"]
    if kind == "operator":
        return x["x"] + kappa ** 2 * x["b"] * _Operator(n, kappa, case["order"])(x["x"])
    if kind == "receivers":
        E = _exact_points(n, kappa, x["xy"])
        return {"field": (x["sigma"].reshape(nrhs, -1) @ E.T), "back": (x["g"] @ E.conj()).reshape(nrhs, n, n)}
    if n * n * nrhs > 256 * 256 * 8:
        return None
    e = _exact_solve(n, kappa, case["order"], x["b"], x["u"])
    if kind != "gradient" or e is None:
        return e
    E, K = _exact_points(n, kappa, x["xy"]), _Operator(n, kappa, case["order"])
    field = e["sigma"].reshape(nrhs, -1) @ E.T
    g = ((field - x["data"]) @ E.conj()).reshape(nrhs, n, n)
    grad = torch.zeros_like(x["b"])
    for m in range(nrhs):  # A^H lambda = g; K is complex symmetric, so A^T y = y + kappa^2 K (b y)
        y = _gmres(lambda v: v + kappa ** 2 * K(x["b"] * v), g[m].conj())
        if y is None:
            return None
        grad -= kappa ** 2 * (y * (x["u"][m] + e["u"][m])).real
    return {"field": field, "grad": grad}
