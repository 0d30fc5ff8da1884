"""Timing cases of the scanner: what one pass of a user's program does on one
MI355X, through the package's public entry points.

A case is a dict of plain values.  `kind` names the entry point (a planned
scan, the one-call scan, the allocation-free scan, the y-plane scan, the
obstruction map, a burst of served requests); the rest are sizes and options.
`prepare` draws the physical parameters (masses, subtraction point, poles) from
the seed, over the ranges of the serving trace; `exact` evaluates the same
quadrature on the same contours with plain torch in 64 bits.
"""
from __future__ import annotations

import cmath
import math
import random

import numpy as np
import torch

import paper_1205_0752_amd as gf
from paper_1205_0752_amd import workloads as wl

BOXES = {
    "bench": (-16.0, 8.0, -8.0, 8.0),    # the 1024^2 workloads
    "wide": (-12.0, 6.0, -6.0, 6.0),     # the 2048^2 workloads
    "window": (-8.0, 4.0, -4.0, 4.0),    # the small workload and the serving window
    "paper": (-5.0, 5.0, -5.0, 5.0),     # the paper's display box
    "cut": (-12.0, 4.0, 0.0, 0.5),       # a strip above the cut
}
RULES = {"gc2": wl.GC2, "gc1": wl.GC1, "tanh_sinh": wl.TANH_SINH, "gl": wl.GL}

BASE = {"kind": "scan", "box": "bench", "n_re": 256, "n_im": 256, "n_r": 128, "n_a": 64,
        "n_arc": 16, "fp32c": False, "rule": "gc2", "split": False, "taylor": 0, "dim": 4,
        "masses": "real", "poles1": 0, "poles2": 0, "numerator": False, "lambda2": 1e6,
        "cls": False}


def _case(name=None, **kw):
    c = dict(BASE, **kw)
    if name:
        c = {"name": name, **c}
    return c


def listed():
    return [
        # the smallest call, made once per parameter point of a fit: launch and latency
        _case("one_call_64sq", kind="one_call", box="window", n_re=64, n_im=64, n_r=64, n_a=32,
              lambda2=1e4),
        # the paper's own working size: 128^2 points over +-5, its complex masses,
        # 64 radial nodes and 49 tanh-sinh angular nodes, with the class map it plots
        _case("paper_box_tanh_sinh", box="paper", n_re=128, n_im=128, n_r=64, n_a=49,
              rule="tanh_sinh", masses="paper", cls=True),
        # the large FP64 scan
        _case("large_fp64", n_re=1024, n_im=1024, n_r=256, n_a=128),
        # the large mixed-precision scan
        _case("large_fp32c", n_re=1024, n_im=1024, n_r=512, n_a=256, fp32c=True),
        # the largest: 2048^2 points, a conjugate mass pair, 512 x 256 nodes
        _case("largest_fp64_conj", box="wide", n_re=2048, n_im=2048, n_r=512, n_a=256,
              masses="conj"),
        # a ragged mid-sized window with a higher subtraction, odd angular order
        _case("ragged_taylor2", box="window", n_re=509, n_im=330, n_r=200, n_a=91, taylor=2),
        # a fine strip over the cut, where the split radial rule is wanted, in D = 4
        _case("cut_strip_split", box="cut", n_re=1500, n_im=47, n_r=256, n_a=256, split=True),
        # pole-sum propagators: a conjugate pair on one leg, two real poles on the other
        _case("pole_sum", n_re=512, n_im=512, n_r=256, n_a=128, poles1=2, poles2=2),
        # recorded or allocation-free use: tables generated on the device by each call
        _case("allocation_free", kind="noalloc", box="window", n_re=200, n_im=150, n_r=256, n_a=96),
        # the y-plane picture at fixed x (Fig. 1): the subtracted integrand
        _case("y_plane", kind="yscan", n_re=1024, n_im=1024, n_a=128),
        # the region map (Fig. 2) of the large box
        _case("obstruction_map", kind="obstruction", n_re=1024, n_im=1024, samples=4096),
        # a burst of mixed requests to the server, submitted together and read back
        _case("served_burst", kind="serve", requests=40, trace=0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


MAX_EVALS = 3e11  # the largest listed case has 5.7e11


def draw(rng):
    k = rng.random()
    if k < 0.08:
        return _case(kind="serve", requests=rng.randint(6, 40), trace=rng.randrange(1 << 20))
    if k < 0.16:
        return _case(kind="yscan", n_re=_log_int(rng, 64, 2048), n_im=_log_int(rng, 64, 2048),
                     n_a=_log_int(rng, 32, 512), rule=rng.choice(["gc2", "gc2", "tanh_sinh"]),
                     masses=rng.choice(["real", "conj"]))
    if k < 0.26:
        return _case(kind="obstruction", box=rng.choice(["bench", "window", "wide", "paper"]),
                     n_re=_log_int(rng, 64, 1024), n_im=_log_int(rng, 64, 1024),
                     samples=_log_int(rng, 256, 8192), masses=rng.choice(["real", "conj"]))
    c = _case(kind="scan" if k < 0.72 else "one_call" if k < 0.86 else "noalloc",
              box=rng.choice(["bench", "wide", "window", "paper", "cut"]),
              n_r=_log_int(rng, 32, 512), n_a=_log_int(rng, 32, 512), n_arc=rng.randint(8, 32),
              fp32c=rng.random() < 0.4, masses=rng.choice(["real", "real", "conj"]),
              rule=rng.choice(["gc2", "gc2", "gc2", "tanh_sinh", "gc1", "gl"]))
    o = rng.random()
    if o < 0.12:
        c["taylor"] = rng.randint(1, 4)
    elif o < 0.24:
        c["split"] = True
        c["n_r"] = 4 * max(8, c["n_r"] // 4)
    elif o < 0.34:
        c["dim"], c["masses"] = rng.choice([2, 3]), "real"
    elif o < 0.50 and c["kind"] == "scan":
        c["poles1"], c["poles2"] = rng.randint(1, 3), rng.randint(1, 3)
        c["numerator"] = rng.random() < 0.3
        if c["numerator"]:  # FP32C is for numerators whose subtracted value stays near the sums
            c["fp32c"] = False
    most = MAX_EVALS / ((c["n_r"] + c["n_arc"]) * c["n_a"] * max(1, c["poles1"]))
    hi = min(2048.0, math.sqrt(most))
    c["n_re"], c["n_im"] = _log_int(rng, 16, hi), _log_int(rng, 16, hi)
    if c["masses"] != "real" or c["box"] != "cut":
        c["n_im"] += c["n_im"] % 2  # no row on the real axis, where real masses have no contour
    c["cls"] = c["kind"] == "scan" and rng.random() < 0.3
    return c


# ---- inputs ---------------------------------------------------------------

def _inputs(case, seed):
    """Parameters, propagators, quadrature and grid of a case, from the seed."""
    rng = random.Random(seed * 1000003 + 17)
    kind = case["masses"]
    if kind == "conj":
        m1 = complex(rng.uniform(0.25, 4.0), rng.uniform(0.1, 1.0))
        m2 = m1.conjugate()
    elif kind == "paper":
        m2 = complex(0.0, rng.uniform(0.4, 0.6))
        m1 = m2.conjugate()
    else:
        m1, m2 = rng.uniform(0.25, 4.0), rng.uniform(0.25, 4.0)
    mu2 = 0.0 if kind == "paper" else rng.uniform(0.5, 4.0)
    taylor = case["taylor"]
    params = gf.Params(m1, m2, mu2, case["lambda2"], 1.0, taylor, case["dim"])
    props = None
    if case["poles1"]:
        def leg(n, pair):
            got = []
            if pair and n >= 2:
                got += gf.Propagators.conjugate_pair(
                    complex(rng.uniform(0.5, 2.0), rng.uniform(0.3, 1.0)), rng.uniform(0.3, 0.7))
            while len(got) < n:
                got.append((rng.uniform(0.25, 4.0), rng.uniform(0.3, 1.0)))
            return tuple(got)
        num = ()
        if case["numerator"]:
            num = tuple((i, j, complex(rng.uniform(-0.4, 0.4), rng.uniform(-0.2, 0.2)) / 10 ** i)
                        for i in range(2) for j in range(3))
        props = gf.Propagators(leg(case["poles1"], True), leg(case["poles2"], False), num)
    quad = gf.Quadrature(case["n_r"], case["n_a"], case["n_arc"],
                         gf.FP32C if case["fp32c"] else gf.FP64, RULES[case["rule"]],
                         1 if case["split"] else 0)
    grid = gf.Grid(case["n_re"], case["n_im"], *BOXES[case["box"]])
    return params, props, quad, grid, rng


def _yscan_inputs(case, seed):
    """The y-plane scan's parameters, x and y grid."""
    params, _, _, _, rng = _inputs(case, seed)
    x = complex(rng.uniform(0.5, 4.0), rng.uniform(0.5, 3.0))
    return params, x, gf.Grid(case["n_re"], case["n_im"], -8.0, 8.0, -8.0, 8.0)


def prepare(case, seed):
    kind = case["kind"]
    if kind == "serve":
        # grids and orders of one trace, masses of another; the program keeps the server
        n = case["requests"]
        sizes = wl.serving_trace(n, 4000.0, seed=case["trace"])
        reqs = [(a.params, b.grid, b.quad)
                for a, b in zip(wl.serving_trace(n, 4000.0, seed=seed), sizes)]
        return {"case": case, "reqs": reqs, "server": gf.Server(budget_bytes=512 << 20)}
    params, props, quad, grid, _ = _inputs(case, seed)
    s = {"case": case, "params": params, "quad": quad, "grid": grid}
    if kind == "yscan":
        _, s["x"], s["grid"] = _yscan_inputs(case, seed)
    if kind in ("scan", "yscan"):
        s["plan"] = gf.Plan(params, quad, props)
    if kind == "obstruction":
        s["out"] = torch.empty((grid.n_im, grid.n_re), dtype=torch.uint8, device="cuda")
    else:
        s["out"] = gf.empty_result(s["grid"])
    if case["cls"]:
        s["cls"] = torch.empty((grid.n_im, grid.n_re), dtype=torch.int8, device="cuda")
    return s


def run(s):
    case = s["case"]
    kind = case["kind"]
    if kind == "scan":
        gf.scan_plan(s["plan"], s["grid"], s["out"], s.get("cls"))
        return {"g": s["out"], "cls": s["cls"]} if case["cls"] else s["out"]
    if kind == "one_call":
        return gf.scan(s["params"], s["grid"], s["quad"], s["out"])
    if kind == "noalloc":
        return gf.scan_noalloc(s["params"], s["grid"], s["quad"], s["out"])
    if kind == "yscan":
        return gf.yscan_plan(s["plan"], s["x"], s["grid"], gf.YSCAN_INTEGRAND, s["out"])
    if kind == "obstruction":
        return gf.obstruction_map(s["params"], s["grid"], case["samples"], s["out"])
    srv = s["server"]
    tickets = [srv.submit(*r) for r in s["reqs"]]
    got = {}
    while len(got) < len(tickets):
        t = srv.wait_any(30000.0)
        if t is None:
            raise RuntimeError("a request did not finish")
        got[t] = srv.result(t)
        srv.release(t)
    return [got[t] for t in tickets]


FLOPS_PER_EVAL = 6.5  # one folded node pair, 13 flops, is two evaluations


def work(case):
    """Points are written once, tables read once; evaluations at the folded
    pair's flops.  The obstruction map: a contour class and the roots of its
    three contour parts per point, with a 40-step bisection."""
    kind = case["kind"]
    if kind == "serve":
        # means of the trace: side^2 = 91,520 points, both orders 198.4, 16 arc nodes
        per = 91520.0
        return {"bytes": case["requests"] * per * 16.0,
                "flops": case["requests"] * per * (198.4 + 16.0) * 198.4 * FLOPS_PER_EVAL}
    n = case["n_re"] * case["n_im"]
    if kind == "obstruction":
        return {"bytes": float(n), "flops": n * 1500.0}
    tables = 8.0 * (2 * case["n_r"] + case["n_a"] + 2 * case["n_arc"])
    if kind == "yscan":
        return {"bytes": 16.0 * n + 8.0 * case["n_a"],
                "flops": n * 2.0 * case["n_a"] * FLOPS_PER_EVAL}
    evals = n * float(case["n_r"] + case["n_arc"]) * case["n_a"] * max(1, case["poles1"])
    return {"bytes": 16.0 * n + tables + (n if case["cls"] else 0), "flops": evals * FLOPS_PER_EVAL}


# ---- the same quadrature in plain torch, 64 bits ----------------------------

EXACT_EVALS = 2e11  # above this the plain evaluation takes too long


def _gauss_legendre(n):
    x, _ = np.polynomial.legendre.leggauss(n)
    for _ in range(3):  # polish
        p0, p1 = np.ones_like(x), x.copy()
        for k in range(1, n):
            p0, p1 = p1, ((2 * k + 1) * x * p1 - k * p0) / (k + 1)
        if n == 1:
            p0, p1 = np.ones_like(x), x
        dp = n * (p0 - x * p1) / (1.0 - x * x)
        x = x - p1 / dp
    return x, 2.0 / ((1.0 - x * x) * dp * dp)


def _angular(n, rule, dim):
    """Nodes z > 0 with doubled weights, and the weight of z = 0 (odd n)."""
    norm = {2: math.pi, 3: 2.0, 4: math.pi / 2}[dim]
    if rule == "gc2":
        th = np.arange(1, n + 1) * math.pi / (n + 1)
        z, w = np.cos(th), math.pi / (n + 1) * np.sin(th) ** (dim - 2) / norm
    elif rule == "gc1":
        th = (2 * np.arange(1, n + 1) - 1) * math.pi / (2 * n)
        z, w = np.cos(th), math.pi / n * np.sin(th) ** (dim - 2) / norm
    elif rule == "gl":
        z, g = _gauss_legendre(n)
        z, w = z[::-1], g[::-1] * (1 - z * z) ** ((dim - 3) / 2) / norm
    else:
        tmax = {4: 3.0, 3: 3.5, 2: 4.0}[dim]
        h = 2 * tmax / (n - 1)
        t = (n - 1) / 2 * h - np.arange(n) * h
        u = math.pi / 2 * np.sinh(t)
        z, w = np.tanh(u), h * math.pi / 2 * np.cosh(t) / np.cosh(u) ** (dim - 1) / norm
    half = n // 2
    return z[:half] ** 2, 2 * w[:half], float(w[half]) if n % 2 else 0.0


def _swept(phi, b):
    return np.where(phi > 0, (b > 0) & (b < phi), (b <= 0) & (b > phi))


def _bad_ray(m):
    return math.pi if m.imag == 0 else math.atan2(-m.imag, -m.real)


def _classes(x, m1, m2, mirror_ok):
    """Contour class of every x: R 0, Y 1, YRES 2, MIRROR 3, SINGULAR 4, LONG 5,
    and whether the real axis is valid there."""
    b1, b2 = [_bad_ray(m) for m in m1], [_bad_ray(m) for m in m2]
    phi = np.arctan2(x.imag, x.real)
    v, vstar = np.abs(np.sqrt(x).imag), min(cmath.sqrt(m).real for m in m1)
    past1, past2 = np.zeros(x.shape, bool), np.zeros(x.shape, bool)
    delta = np.full(x.shape, math.pi)
    for bs, past in ((b1, past1), (b2, past2)):
        for b in bs:
            past |= _swept(phi, b)
            d = np.abs(phi - b)
            delta = np.minimum(delta, np.where(d > math.pi, 2 * math.pi - d, d))
    hi = min([b for b in b1 + b2 if b > 0], default=math.pi)
    lo = max([b for b in b1 + b2 if b <= 0], default=-math.pi)
    rot = np.full(x.shape, 5)
    rot[past1 & ~past2 & mirror_ok] = 3
    rot[past2 & ~past1] = 2
    rot[delta == 0.0] = 4
    rot[(phi > lo) & (phi < hi)] = 1
    valid = v < vstar
    near = (v < 0.25 * vstar) | (1.0 - v / vstar >= 0.45 * delta) | (rot >= 4)
    return np.where(valid & near, 0, rot), valid


def _split_nodes(x, m1, m2, T, lam2, gx, gw):
    """r and dt-weight of the split rule, [4 m] x points: four pieces cut at the
    near-singular radii of each x."""
    sx, sm = np.sqrt(x), cmath.sqrt(-m1)
    cand = np.stack([np.abs(sx + sm) ** 2, np.abs(sx - sm) ** 2, np.full(x.shape, abs(m2))])
    b = np.full((5,) + x.shape, np.inf)
    b[0], b[1] = 0.0, T
    nb = np.full(x.shape, 2)
    cols = np.arange(x.size)
    for k in range(3):
        ok = (cand[k] > 0) & (cand[k] < lam2)
        t = np.log1p(np.where(ok, cand[k], 1.0))
        for q in range(5):
            ok &= ~((q < nb) & (np.abs(np.where(np.isinf(b[q]), 1e300, b[q]) - t) <= 1e-9 * T))
        b[nb[ok], cols[ok]] = t[ok]
        b = np.sort(b, axis=0)
        nb = nb + ok
    for _ in range(3):
        todo = nb < 5
        wide = np.zeros(x.shape, int)
        for i in range(1, 4):
            gap = np.where(i < nb - 1, b[i + 1] - b[i], -1.0)
            best = b[wide + 1, cols] - b[wide, cols]
            wide = np.where(gap > best + 1e-12 * T, i, wide)
        mid = 0.5 * (b[wide, cols] + b[wide + 1, cols])
        b[nb[todo], cols[todo]] = mid[todo]
        b = np.sort(b, axis=0)
        nb = nb + todo
    h = 0.5 * (b[1:] - b[:-1])
    r = np.expm1(h[:, None] * (gx[None, :, None] + 1.0) + b[:-1][:, None])
    w = h[:, None] * gw[None, :, None] * (1.0 + r)
    return r.reshape(-1, x.size), w.reshape(-1, x.size)


class _Sum:
    """Contour sums of one integrand over sets of points (numpy in and out, the
    angular sums in torch on the GPU)."""

    def __init__(self, case, params, props):
        self.dim, self.lam2 = params.dimension, params.lambda2
        self.T = math.log1p(self.lam2)
        self.split = case["split"]
        self.m1 = [(complex(m), complex(c)) for m, c in (props.poles1 if props else ((params.m1sq, 1.0),))]
        self.m2 = [(complex(m), complex(c)) for m, c in (props.poles2 if props else ((params.m2sq, 1.0),))]
        self.num = {(i, j): complex(c) for i, j, c in (props.numerator if props else ())}
        s, w, self.wmid = _angular(case["n_a"], case["rule"], self.dim)
        self.s_np, self.w_np = s, w
        dev = torch.device("cuda" if torch.cuda.is_available() else "cpu")
        self.dev = dev
        self.s = torch.from_numpy(np.ascontiguousarray(s)).to(dev)
        self.w = torch.from_numpy(np.stack([w, w * s], 1)).to(dev, torch.complex128)
        if self.split:
            self.gx, self.gw = _gauss_legendre(case["n_r"] // 4)
        else:
            gx, gw = _gauss_legendre(case["n_r"])
            r = np.expm1(0.5 * self.T * (gx + 1.0))
            self.r, self.rw = r, 0.5 * self.T * gw * (1.0 + r)
        self.ax, self.aw = _gauss_legendre(case["n_arc"])

    def term(self, x, y, a, weight):
        """weight * P2(y) * <N / (x + y + m1_a^2 - 2 sqrt(x y) z)> (torch, points)."""
        U, V2 = x + y + self.m1[a][0], 4.0 * x * y
        A, S1 = torch.empty_like(U), torch.empty_like(U)
        step = max(1, (1 << 24) // max(1, self.s.numel()))
        for i in range(0, U.numel(), step):
            u, v2 = U[i:i + step], V2[i:i + step]
            both = ((u * u)[:, None] - v2[:, None] * self.s[None, :]).reciprocal() @ self.w
            A[i:i + step], S1[i:i + step] = u * both[:, 0], both[:, 1]
        if self.wmid:
            A = A + self.wmid / U
        if self.num:
            N = [sum(self.num.get((i, j), 0.0) * y ** i for i in range(3)) + 0.0 * y for j in range(3)]
            A = N[0] * A + N[1] * (0.5 * V2 * S1) + N[2] * (0.25 * V2 * U * S1)
        return self.m1[a][1] * weight * A

    def p2(self, y):
        return sum(c / (y + m) for m, c in self.m2)

    def measure(self, y, sqrt_y):
        return y if self.dim == 4 else sqrt_y if self.dim == 3 else torch.ones_like(y)

    def contour(self, x, ray):
        """Sum along the straight part to angle `ray` (0: real axis), then, with
        ray, the closing arcs and the swept k-leg residues of each (p-k) pole."""
        tx = torch.from_numpy(x).to(self.dev)
        phi = np.arctan2(x.imag, x.real) if ray else np.zeros(x.shape)
        tphi = torch.from_numpy(phi).to(self.dev)
        e, half = torch.polar(torch.ones_like(tphi), tphi), torch.polar(torch.ones_like(tphi), 0.5 * tphi)
        total = torch.zeros_like(tx)
        if self.split:
            r, w = _split_nodes(x, self.m1[0][0], self.m2[0][0], self.T, self.lam2, self.gx, self.gw)
            nodes = [(torch.from_numpy(r[k]).to(self.dev), torch.from_numpy(w[k]).to(self.dev))
                     for k in range(r.shape[0])]
        else:
            nodes = [(torch.full_like(tphi, r), torch.full_like(tphi, w)) for r, w in zip(self.r, self.rw)]
        for r, w in nodes:
            y = e * r
            q = self.measure(y, half * r.sqrt()) * e * w * self.p2(y)
            for a in range(len(self.m1)):
                total = total + self.term(tx, y, a, q)
        if not ray:
            return total.cpu().numpy()
        b2 = [_bad_ray(m) for m, _ in self.m2]
        for a, (m, _) in enumerate(self.m1):
            # the long way round where this pole's bad ray would be swept
            lng = _swept(phi, _bad_ray(m))
            L = np.where(phi > 0, 2 * math.pi, -2 * math.pi) - phi
            for xi, wa in zip(self.ax, self.aw):
                psi = np.where(lng, phi + 0.5 * L * (1 + xi), 0.5 * phi * (1 - xi))
                h = np.where(lng, 0.5 * L * wa, -0.5 * phi * wa)
                psi, h = torch.from_numpy(psi).to(self.dev), torch.from_numpy(h).to(self.dev)
                y = self.lam2 * torch.polar(torch.ones_like(psi), psi)
                f = self.measure(y, math.sqrt(self.lam2) * torch.polar(torch.ones_like(psi), 0.5 * psi))
                total = total + self.term(tx, y, a, 1j * y * h * f * self.p2(y))
            for b, (m2, c2) in enumerate(self.m2):
                sw = _swept(phi, b2[b])
                sign = np.where(lng, np.where(sw, 0.0, -np.sign(phi)), np.where(sw, np.sign(phi), 0.0))
                if not np.any(sign):
                    continue
                y0 = torch.full_like(tx, -m2)
                f = self.measure(y0, y0.sqrt())
                wt = torch.from_numpy(2j * math.pi * sign).to(self.dev) * c2 * f
                val = self.term(tx, y0, a, wt)
                total = total + torch.where(torch.from_numpy(sign != 0.0).to(self.dev), val, 0.0)
        return total.cpu().numpy()

    def taylor(self, mu2, n):
        """K_0..K_n of the real-axis sum about mu2: power series of each pair's
        w U / (U^2 - 4 x y s) in x - mu2."""
        K = np.zeros(n + 1, complex)
        K[0] = self.contour(np.array([complex(mu2)]), False)[0]
        if n == 0:
            return K
        if self.split:
            r, w = _split_nodes(np.array([complex(mu2)]), self.m1[0][0], self.m2[0][0], self.T,
                                self.lam2, self.gx, self.gw)
            r, w = r[:, 0], w[:, 0]
        else:
            r, w = self.r, self.rw
        om = w * (r if self.dim == 4 else np.sqrt(r) if self.dim == 3 else 1.0)
        om = om * sum(c / (r + m) for m, c in self.m2)
        s, w2 = self.s_np[None, :], self.w_np[None, :]
        for m, c in self.m1:
            U, y = (mu2 + r + m)[:, None], r[:, None]
            D0, D1 = U * U - 4 * mu2 * y * s, 2 * U - 4 * y * s
            q2, q1 = 0.0, w2 * U / D0
            mid = self.wmid / U[:, 0]
            for i in range(1, n + 1):
                q = ((w2 if i == 1 else 0.0) - D1 * q1 - q2) / D0
                mid = -mid / U[:, 0]
                K[i] += c * np.sum(om * (q.sum(1) + mid))
                q2, q1 = q1, q
        return K


def _exact_scan(case, seed):
    params, props, quad, grid, _ = _inputs(case, seed)
    S = _Sum(case, params, props)
    a, b = np.arange(grid.n_re) + 0.5, np.arange(grid.n_im) + 0.5
    re = a * ((grid.re_hi - grid.re_lo) / grid.n_re) + grid.re_lo
    im = b * ((grid.im_hi - grid.im_lo) / grid.n_im) + grid.im_lo
    x = (re[None, :] + 1j * im[:, None]).ravel()
    m1, m2 = [m for m, _ in S.m1], [m for m, _ in S.m2]
    key = lambda ps, f: sorted((f(m).real, f(m).imag, f(c).real, f(c).imag) for m, c in ps)  # noqa: E731
    one, con = (lambda v: v + 0), (lambda v: v.conjugate() + 0)
    same = key(S.m1, con) == key(S.m1, one) and key(S.m2, con) == key(S.m2, one)
    swap = key(S.m1, con) == key(S.m2, one) and key(S.m2, con) == key(S.m1, one)
    mirror = (same and all(c.imag == 0 for c in S.num.values())) if S.num else (same or swap)
    cls, valid = _classes(x, m1, m2, mirror)
    flip = np.zeros(x.shape, bool)
    at = cls == 3
    if at.any():
        back, _ = _classes(x[at].conj(), m1, m2, mirror)
        own = back < 3
        flip[np.nonzero(at)[0][own]] = True
        cls[np.nonzero(at)[0][~own]] = np.where(valid[at][~own], 0, 5)
    ev = np.where(flip, x.conj(), x)
    real = cls == 0
    if flip.any():
        real[flip] = _classes(ev[flip], m1, m2, mirror)[0] == 0
    g = np.full(x.shape, complex(math.nan, math.nan))
    n = params.taylor_order
    K = S.taylor(params.mu2, max(n, 0))
    for ray, sel in ((False, real & (cls != 4)), (True, ~real & (cls != 4))):
        if sel.any():
            d = ev[sel] - params.mu2
            g[sel] = S.contour(ev[sel], ray) - sum(K[i] * d ** i for i in range(n + 1))
    g = params.scale * np.where(flip, g.conj(), g)
    return g.reshape(grid.n_im, grid.n_re)


def exact(case, seed):
    kind = case["kind"]
    if kind in ("serve", "obstruction"):
        return None
    if kind == "yscan":
        params, x, grid = _yscan_inputs(case, seed)
        S = _Sum(case, params, None)
        re = (np.arange(grid.n_re) + 0.5) * ((grid.re_hi - grid.re_lo) / grid.n_re) + grid.re_lo
        im = (np.arange(grid.n_im) + 0.5) * ((grid.im_hi - grid.im_lo) / grid.n_im) + grid.im_lo
        y = torch.from_numpy((re[None, :] + 1j * im[:, None]).ravel()).to(S.dev)
        q = y * S.p2(y)
        got = S.term(torch.full_like(y, x), y, 0, q) - S.term(torch.full_like(y, params.mu2), y, 0, q)
        return got.cpu().numpy().reshape(grid.n_im, grid.n_re)
    evals = (float(case["n_re"]) * case["n_im"] * (case["n_r"] + case["n_arc"]) * case["n_a"]
             * max(1, case["poles1"]))
    if evals > EXACT_EVALS:
        return None
    g = _exact_scan(case, seed)
    return {"g": g, "cls": None} if case["cls"] else g

