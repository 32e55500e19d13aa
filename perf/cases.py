"""Performance cases: what a user of the library has it do, over the range of sizes,
pixel kinds, gain modes, precisions and calls that the workloads of this repository span.

A case is a dict of plain values.  ``prepare`` makes what a user's program holds before a
call (positions, baselines, a sky, data, the plan or the server), ``run`` is one pass
through the public Python API, ``exact`` the same outputs in float64 from the closed form
of every matrix entry, without the library.
"""
import math
from types import SimpleNamespace

import numpy as np
import torch

from paper_1310_2078_amd import sl1m
from paper_1310_2078_amd import workloads as W

FWHM = 0.4        # power-beam width of the cases with gains (radians)


def listed():
    return [
        # The smallest operator call (a 32 x 32 snapshot image): launches and latency.
        _op("forward_small", "forward", 32, 2_000, extent=0.05, array=False),
        # A whole small deconvolution, step constant included: 30 power steps, 100
        # iterations and the objective; a user runs thousands of these over channels.
        dict(_op("solve_small", "solve", 32, 2_000, extent=0.05, array=False), iters=100),
        # One application of each operator on the medium image (256 x 256 wide field,
        # 128 antennas, 12 snapshots): what any outer iteration of a user's own is made of.
        _op("operators_medium", "operators", 256, 97_536, extent=0.3),
        # A checkpointed piece of a medium solve: 8 FISTA iterations from a saved state.
        dict(_op("fista_medium", "fista", 256, 97_536, extent=0.3), iters=8),
        # Stokes I, Q, U, V through one matrix at the medium size.
        _op("stokes4_medium", "operators", 256, 97_536, extent=0.3, sides=4),
        # Eight planes at once in the float16 matrix-core precision.
        _op("f16_eight_medium", "operators", 256, 97_536, extent=0.3, sides=8,
            precision="mfma_f16"),
        # The largest: a 1024 x 1024 image with three layers of wide Gaussian pixels, 256
        # antennas, flagged records, gains and a beam; each operator on its own.
        _op("forward_large", "forward", 1024, 409_600, extent=0.35, pixels="layers", gains=True),
        _op("adjoint_large", "adjoint", 1024, 409_600, extent=0.35, pixels="layers", gains=True),
        # One request of the channel stream: Gaussian pixels on a row-major grid cut off
        # mid-row (odd sizes); its dirty image and the model visibilities of a sky.
        _op("request_gauss", "request", 300, 100_003, extent=0.05, array=False,
            pixels="truncated", gauss=True),
        # A level of the adaptive refinement: cells of four sizes at scattered places (no
        # grid to exploit), gains on.
        _op("refine_cells", "operators", 192, 102_400, extent=0.35, pixels="cells", gains=True),
        # The float64 plan that results are checked with; every antenna with a beam of its
        # own, an odd image.
        _op("float64_check", "operators", 45, 20_011, extent=0.25, gains=True, beams=True,
            precision="fp64"),
        # The server: eight requests of mixed size and kind, submitted together.
        dict(_op("serve_mix", "serve", 64, 10_000, extent=0.05, array=False), iters=20,
             requests=8),
    ]


def draw(rng):
    """One more case of the same ranges."""
    def log(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    path = rng.choice(["forward", "adjoint", "operators", "operators", "solve", "fista", "request",
                       "serve"])
    if path == "serve":
        return dict(_op(None, path, rng.randint(48, 90), log(6_000, 16_000), extent=0.05,
                        array=False), iters=rng.randint(8, 24), requests=rng.randint(4, 9))
    if path == "solve":
        return dict(_op(None, path, rng.randint(32, 72), log(2_000, 9_000),
                        extent=rng.choice([0.05, 0.1]), array=False), iters=rng.randint(20, 100))
    if path == "fista":
        return dict(_op(None, path, rng.randint(48, 256), log(8_000, 97_536),
                        extent=rng.uniform(0.05, 0.3)), iters=rng.randint(3, 8))
    if path == "request":
        return _op(None, path, log(64, 512), log(10_000, 200_000), extent=0.05, array=False,
                   pixels="truncated", gauss=rng.random() < 0.5)
    pixels = rng.choice(["grid", "grid", "layers", "cells", "truncated"])
    sides = rng.choice([1, 1, 2, 4, 8]) if pixels == "grid" and path == "operators" else 1
    precision = rng.choice(["fp32", "fp32", "fp32", "mfma_f16", "fp64"])
    if pixels != "grid" or (precision == "mfma_f16" and sides < 4):
        precision = "fp32"
    if precision == "fp64":
        return _op(None, path, rng.randint(33, 80), log(5_000, 40_000),
                   extent=rng.uniform(0.05, 0.3), gains=True, beams=rng.random() < 0.5,
                   precision=precision)
    if pixels == "cells":
        return _op(None, path, rng.randint(64, 200), log(10_000, 150_000), extent=0.35,
                   pixels=pixels, gains=True)
    if pixels == "layers":
        side = 8 * rng.randint(12, 80)
        return _op(None, path, side, log(10_000, 200_000), extent=0.35 * side / 1024,
                   pixels=pixels, gains=True)
    return _op(None, path, log(32, 640 if sides == 1 else 300), log(2_000, 200_000),
               extent=rng.uniform(0.05, 0.35), array=rng.random() < 0.7, pixels=pixels,
               gains=precision == "fp32" and rng.random() < 0.4, precision=precision, sides=sides)


def _op(name, path, side, vis, extent, array=True, pixels="grid", gauss=False, gains=False,
        beams=False, precision="fp32", sides=1):
    """array: baselines of a random 3 km array over six hours at 150 MHz, else (u, v) in a
    500-wavelength disk; beams: a beam width per antenna instead of one for all."""
    c = dict(path=path, side=int(side), vis=int(vis), extent=float(extent), array=bool(array),
             pixels=pixels, gauss=bool(gauss), gains=bool(gains), beams=bool(beams),
             precision=precision, sides=int(sides))
    return c if name is None else dict(name=name, **c)


# ---------------------------------------------------------------------------
# inputs
# ---------------------------------------------------------------------------

def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _pixels(c, rng):
    """l, m, sigma, kind of a case's pixels."""
    side, ext = c["side"], c["extent"]
    l, m, d = W.grid_pixels(side, ext)
    sigma, kind = np.zeros(l.size), np.zeros(l.size, np.uint8)
    if c["pixels"] == "layers":
        # a delta grid, then wide Gaussian layers of 2, 4 and 8 spacings
        parts = [(l, m, sigma, kind)]
        for f in (2, 4, 8):
            lg, mg, _ = W.grid_pixels(side // f, ext)
            parts.append((lg, mg, np.full(lg.size, f * d),
                          np.full(lg.size, W.PIX_GAUSS_WIDE, np.uint8)))
        l, m, sigma, kind = (np.concatenate([p[i] for p in parts]) for i in range(4))
    elif c["pixels"] == "truncated":
        n = side * (side - 1) - side // 3      # the last row is cut off
        l, m, sigma, kind = l[:n], m[:n], sigma[:n], kind[:n]
    elif c["pixels"] == "cells":
        # a refinement level: of every 8 cells five stay coarse Gaussians of three sizes,
        # the others are delta pixels, shifted off the grid as refined children are
        which = rng.integers(0, 8, l.size)
        size = np.where(which < 2, 4.0, np.where(which < 4, 2.0, np.where(which < 5, 1.0, 0.0)))
        sigma = 0.5 * size * d
        kind = np.where(size > 0, W.PIX_GAUSS_WIDE, W.PIX_DELTA).astype(np.uint8)
        l = l + rng.integers(-4, 5, l.size) * (d / 8)
        m = m + rng.integers(-4, 5, l.size) * (d / 8)
    if c["gauss"]:
        sigma, kind = np.full(l.size, 2.0 * d), np.full(l.size, W.PIX_GAUSS_WIDE, np.uint8)
    return l, m, sigma, kind


def _inputs(c, seed):
    """The problem of a case as host arrays (a workload-like object), from the seed alone."""
    rng = np.random.default_rng(seed)
    l, m, sigma, kind = _pixels(c, rng)
    nv = c["vis"]
    ap = aq = gain = fwhm = None
    if c["array"]:
        snaps = 13 if c["pixels"] == "layers" else 12
        n_ant = int(math.ceil(0.5 + math.sqrt(0.25 + 2.0 * nv / snaps)))
        e, n, up = W.random_array_enu(rng, n_ant, 3000.0, 20.0)
        p, q = W.baseline_pairs(n_ant)
        u, v, w, ap, aq = W.enu_to_uvw(e, n, up, p, q, W.hour_angles(snaps), math.radians(-27.0),
                                       math.radians(-30.0), W.SPEED_OF_LIGHT / 150e6)
        keep = np.sort(rng.permutation(u.size)[:nv])      # the others are flagged
        u, v, w, ap, aq = u[keep], v[keep], w[keep], ap[keep], aq[keep]
    else:
        u, v, w = W.disk_uvw(rng, nv, 500.0, 50.0)
        n_ant = 32
    if c["gains"]:
        if ap is None:
            ap = rng.integers(0, n_ant, nv).astype(np.int32)
            aq = ((ap + rng.integers(1, n_ant, nv)) % n_ant).astype(np.int32)
        gain = (1.0 + 0.05 * rng.standard_normal(n_ant)) * np.exp(
            0.05j * rng.standard_normal(n_ant))
        fwhm = rng.uniform(0.3, 0.6, n_ant) if c["beams"] else np.full(n_ant, FWHM)
    else:
        ap = aq = None
    return SimpleNamespace(l=l, m=m, sigma=sigma, kind=kind, u=u, v=v, w=w, ant_p=ap, ant_q=aq,
                           ant_gain=gain, ant_fwhm=fwhm, rng=rng, n_pix=l.size, n_vis=nv)


def _sky(c, p):
    """Images [sides, n_pix] (float32 values): point sources over a faint background."""
    x = 1e-3 * np.abs(p.rng.standard_normal((c["sides"], p.n_pix)))
    src = p.rng.choice(p.n_pix, min(200, p.n_pix // 8), replace=False)
    x[:, src] += W.power_law_flux(p.rng, src.size)
    x[1:] *= 0.1
    return x.astype(np.float32)


def _residual(c, p):
    """Residual visibilities [sides, n_vis] (complex64 values): a few sources and noise."""
    r = np.stack([W.complex_noise(p.rng, p.n_vis, 0.3) for _ in range(c["sides"])])
    ls, ms = p.rng.uniform(-0.5, 0.5, (2, 3)) * c["extent"]
    for a, b in zip(ls, ms):
        nu = -(a * a + b * b) / (1.0 + math.sqrt(1.0 - a * a - b * b))
        r += np.exp(-2j * np.pi * (p.u * a + p.v * b + p.w * nu))
    return r.astype(np.complex64)


def _data(c, p):
    """Noisy data of five delta sources on pixels, and the problem's lambda."""
    dev = _device()
    src = p.rng.choice(p.n_pix, 5, replace=False)
    flux = p.rng.uniform(0.5, 2.0, 5)
    u, v, w = (torch.as_tensor(t, device=dev) for t in (p.u, p.v, p.w))
    vis = torch.zeros(p.n_vis, dtype=torch.complex128, device=dev)
    for j, f in zip(src, flux):
        n = math.sqrt(1.0 - p.l[j] ** 2 - p.m[j] ** 2)
        t = 2.0 * math.pi * torch.frac(u * p.l[j] + v * p.m[j] + w * (n - 1.0))
        vis += (f / n) * torch.polar(torch.ones_like(t), -t)
    vis += torch.as_tensor(W.complex_noise(p.rng, p.n_vis, 0.01), device=dev)
    return vis.to(torch.complex64), 3.0 * 0.01 * math.sqrt(p.n_vis)


def _step_constant(c, p):
    """A step constant for the cases that start from a saved one, a little above the largest
    eigenvalue: on a grid of n pixels of spacing d that is about n times the largest number
    of baselines in a cell of the uv plane (side 1 / (d sqrt(n)), baselines modulo 1 / d)."""
    d = 2.0 * c["extent"] / c["side"]
    iu, iv = (np.floor(c["side"] * np.mod(t * d, 1.0)).astype(np.int64) % c["side"]
              for t in (p.u, p.v))
    return 1.5 * float(np.bincount(iu * c["side"] + iv).max()) * p.n_pix


def _requests(c, seed):
    """The server's requests: sizes from half to the whole of the case's, every second one
    with Gaussian pixels, row-major grids cut off mid-row."""
    out = []
    for k in range(c["requests"]):
        rng = np.random.default_rng(10_000 + k)          # sizes belong to the case
        side = int(c["side"] * rng.uniform(0.6, 1.0))
        q = dict(c, path="request", side=side, vis=int(c["vis"] * rng.uniform(0.5, 1.0)),
                 pixels="truncated", gauss=k % 2 == 1)
        p = _inputs(q, seed * 64 + k)
        vis, _ = _data(q, p)
        out.append((p, vis, 0.01))
    return out


# ---------------------------------------------------------------------------
# the passes
# ---------------------------------------------------------------------------

def prepare(case, seed):
    c = dict(case)
    dev = torch.device("cuda")
    s = SimpleNamespace(c=c)
    if c["path"] == "serve":
        s.requests = _requests(c, seed)
        s.server = sl1m.Server(1 << 30, max_slots=c["requests"], round_budget=3e10)
        return s
    p = _inputs(c, seed)
    s.plan = sl1m.Plan.from_workload(p, precision=c["precision"], max_rhs=c["sides"])
    real, cplx = s.plan.rdtype, s.plan.cdtype
    if c["path"] in ("forward", "operators", "request"):
        s.x = torch.as_tensor(_sky(c, p), device=dev).to(real)
    if c["path"] in ("adjoint", "operators", "request"):
        s.r = torch.as_tensor(_residual(c, p), device=dev).to(cplx)
    if c["path"] in ("solve", "fista"):
        s.vis, s.lam = _data(c, p)
        s.vis = s.vis.to(cplx)
    if c["path"] == "fista":
        s.L = _step_constant(c, p)
        img = torch.as_tensor(0.1 * _sky(c, p)[0], device=dev).to(real)
        s.state = {"img": img, "y": 1.25 * img, "t": 6.0, "k": 10}
    return s


def run(s):
    c = s.c
    path, many = c["path"], c["sides"] > 1
    if path == "serve":
        tickets = [s.server.submit(p, vis, lam, c["iters"], power_iters=5)
                   for p, vis, lam in s.requests]
        s.server.drain(tickets)
        out = [s.server.result(t) for t in tickets]
        for t in tickets:
            s.server.release(t)
        return out
    if path == "solve":
        img, info = s.plan.solve(s.vis, s.lam, c["iters"])
        return {"image": img, "objective": info["F"], "L": info["L"]}
    if path == "fista":
        img, info, state = s.plan.solve_resume(s.vis, s.lam, c["iters"], s.L, state=s.state)
        return {"image": img, "point": state["y"], "t": state["t"], "objective": info["F"]}
    out = {}
    if path in ("forward", "operators", "request"):
        out["vis"] = s.plan.forward_multi(s.x) if many else s.plan.forward(s.x[0])
    if path in ("adjoint", "operators"):
        out["gradient"] = s.plan.adjoint_multi(s.r) if many else s.plan.adjoint(s.r[0])
    if path == "request":
        out["dirty"] = s.plan.dirty_image(s.r[0])
    return out


# ---------------------------------------------------------------------------
# the work a pass cannot do without
# ---------------------------------------------------------------------------

def _n_pix(c):
    side = c["side"]
    if c["pixels"] == "layers":
        return side * side + sum((side // f) ** 2 for f in (2, 4, 8))
    if c["pixels"] == "truncated":
        return side * (side - 1) - side // 3
    return side * side


def work(case):
    """Applications x (positions, baselines and vectors once) bytes; per application and
    entry one complex multiply-add by a real number or its real part (4 flops)."""
    c = case
    if c["path"] == "serve":
        b = f = 0.0
        for k in range(c["requests"]):
            rng = np.random.default_rng(10_000 + k)
            q = dict(c, path="request", side=int(c["side"] * rng.uniform(0.6, 1.0)),
                     vis=int(c["vis"] * rng.uniform(0.5, 1.0)), pixels="truncated")
            apps = 2 * 5 + 2 * c["iters"] + 1
            b += apps * (20.0 * _n_pix(q) + 32.0 * q["vis"])
            f += apps * 4.0 * _n_pix(q) * q["vis"]
        return {"bytes": b, "flops": f}
    apps = {"forward": 1, "adjoint": 1, "operators": 2, "request": 2,
            "solve": 2 * 30 + 2 * c.get("iters", 0) + 1, "fista": 2 * c.get("iters", 0) + 1}
    n, size = apps[c["path"]], 8.0 if c["precision"] == "fp64" else 4.0
    per = (16.0 + size * c["sides"]) * _n_pix(c) + (24.0 + 2.0 * size * c["sides"]) * c["vis"]
    return {"bytes": n * per, "flops": n * 4.0 * c["sides"] * _n_pix(c) * c["vis"]}


# ---------------------------------------------------------------------------
# the same outputs in float64
# ---------------------------------------------------------------------------

class _Exact:
    """The operator in float64, every entry from its closed form, in blocks of
    visibilities; small matrices are kept."""

    KEEP, BLOCK = 1 << 28, 1 << 26

    def __init__(self, p):
        dev = _device()
        t = lambda a: torch.as_tensor(np.asarray(a, np.float64), device=dev)
        self.l, self.m, self.sigma = t(p.l), t(p.m), t(p.sigma)
        self.u, self.v, self.w = t(p.u), t(p.v), t(p.w)
        self.gauss = bool(np.any(p.kind != 0))
        r2 = self.l ** 2 + self.m ** 2
        n = torch.sqrt(1.0 - r2)
        self.r2, self.nu, self.inv_n = r2, -r2 / (1.0 + n), 1.0 / n
        self.kappa = -(r2 * r2) / (2.0 * (1.0 + n) ** 2)
        self.gain = self.beam = None
        if p.ant_p is not None and p.ant_gain is not None:
            a, b = (torch.as_tensor(i.astype(np.int64), device=dev) for i in (p.ant_p, p.ant_q))
            g = torch.as_tensor(p.ant_gain, device=dev)
            self.gain = g[a] * g[b].conj()
            f = t(p.ant_fwhm)
            self.beam = -2.0 * math.log(2.0) * (1.0 / f[a] ** 2 + 1.0 / f[b] ** 2)
        self.n_pix, self.n_vis = self.l.numel(), self.u.numel()
        self.step = max(1, self.BLOCK // max(1, self.n_pix))
        self.kept = {} if self.n_pix * self.n_vis <= self.KEEP else None

    def block(self, k0):
        """Rows k0 .. of M as (re, im)."""
        if self.kept is not None and k0 in self.kept:
            return self.kept[k0]
        s = slice(k0, min(k0 + self.step, self.n_vis))
        u, v, w = self.u[s, None], self.v[s, None], self.w[s, None]
        if self.gauss:
            s2 = self.sigma ** 2
            q = w * s2
            D = 1.0 / (1.0 + q * q)
            rho2 = u * u + v * v
            nu = torch.where(self.sigma > 0, self.kappa, self.nu)
            th = D * (0.5 * w * (torch.where(self.sigma > 0, self.r2, 0.0 * self.r2) - s2 * s2 * rho2)
                      - u * self.l - v * self.m) - w * nu
            amp = self.inv_n * D * torch.exp(
                -math.pi * s2 * D * ((u - w * self.l) ** 2 + (v - w * self.m) ** 2))
        else:
            th = -(u * self.l + v * self.m + w * self.nu)
            amp, q = self.inv_n.expand_as(th), None
        if self.beam is not None:
            amp = amp * torch.exp(self.beam[s, None] * self.r2)
        th = (2.0 * math.pi) * (th - torch.round(th))
        re, im = amp * torch.cos(th), amp * torch.sin(th)
        if q is not None:
            re, im = re - q * im, im + q * re
        if self.gain is not None:
            g = self.gain[s, None]
            re, im = g.real * re - g.imag * im, g.real * im + g.imag * re
        if self.kept is not None:
            self.kept[k0] = (re, im)
        return re, im

    def forward(self, x):
        """x [R, n_pix] -> [R, n_vis] complex128."""
        rows = []
        for k0 in range(0, self.n_vis, self.step):
            re, im = self.block(k0)
            rows.append(torch.complex(x @ re.T.contiguous(), x @ im.T.contiguous()))
        return torch.cat(rows, 1)

    def adjoint(self, r):
        """r [R, n_vis] complex128 -> [R, n_pix]."""
        g = torch.zeros((r.shape[0], self.n_pix), dtype=torch.float64, device=r.device)
        for k0 in range(0, self.n_vis, self.step):
            re, im = self.block(k0)
            s = slice(k0, k0 + re.shape[0])
            g += r.real[:, s].contiguous() @ re + r.imag[:, s].contiguous() @ im
        return g


def _uniforms(n):
    """The power iteration's start vector: SplitMix64 in counter form, state 0."""
    with np.errstate(over="ignore"):
        z = (np.arange(1, n + 1, dtype=np.uint64)) * np.uint64(0x9E3779B97F4A7C15)
        z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
        z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
        z = z ^ (z >> np.uint64(31))
    return (z >> np.uint64(11)).astype(np.float64) * 2.0 ** -53


def _exact_L(op, steps):
    x = torch.as_tensor(_uniforms(op.n_pix), device=op.l.device)[None]
    x = x / x.norm()
    rq = 0.0
    for _ in range(steps):
        y = op.adjoint(op.forward(x))
        rq = float((x * y).sum())
        x = y / y.norm()
    return 1.01 * rq


def _exact_fista(op, vis, lam, L, iters, img, y, t):
    vis = vis.to(torch.complex128)[None]
    for _ in range(iters):
        z = y - op.adjoint(op.forward(y) - vis) / L
        new = torch.clamp(z - lam / L, min=0.0)
        tn = 0.5 * (1.0 + math.sqrt(1.0 + 4.0 * t * t))
        y = new + ((t - 1.0) / tn) * (new - img)
        img, t = new, tn
    return img, y, t


def _objective(op, vis, lam, img):
    d = op.forward(img) - vis.to(torch.complex128)[None]
    return 0.5 * float((d.real ** 2 + d.imag ** 2).sum()) + lam * float(img.sum())


def exact(case, seed):
    c = dict(case)
    dev = _device()
    if c["path"] == "serve":
        out = []
        for p, vis, lam in _requests(c, seed):
            op = _Exact(p)
            zero = torch.zeros((1, p.n_pix), dtype=torch.float64, device=dev)
            img, _, _ = _exact_fista(op, vis, lam, _exact_L(op, 5), c["iters"], zero, zero, 1.0)
            out.append(img[0])
        return out
    entries = work(c)["flops"] / (4.0 * c["sides"])
    if entries > 2.5e11:
        return None
    p = _inputs(c, seed)
    op = _Exact(p)
    x = r = None
    if c["path"] in ("forward", "operators", "request"):
        x = torch.as_tensor(_sky(c, p), device=dev).to(torch.float64)
    if c["path"] in ("adjoint", "operators", "request"):
        r = torch.as_tensor(_residual(c, p), device=dev).to(torch.complex128)
    if c["path"] in ("solve", "fista"):
        vis, lam = _data(c, p)
        if c["path"] == "solve":
            zero = torch.zeros((1, p.n_pix), dtype=torch.float64, device=dev)
            L = _exact_L(op, 30)
            img, _, _ = _exact_fista(op, vis, lam, L, c["iters"], zero, zero, 1.0)
            return {"image": img[0], "objective": _objective(op, vis, lam, img), "L": L}
        img = torch.as_tensor(0.1 * _sky(c, p), device=dev)
        start, y = img.to(torch.float64), (1.25 * img).to(torch.float64)
        img, y, t = _exact_fista(op, vis, lam, _step_constant(c, p), c["iters"], start, y, 6.0)
        return {"image": img[0], "point": y[0], "t": t, "objective": _objective(op, vis, lam, img)}
    one = c["sides"] == 1
    out = {}
    if x is not None:
        V = op.forward(x)
        out["vis"] = V[0] if one else V
    if r is not None:
        g = op.adjoint(r)
        if c["path"] == "request":
            out["dirty"] = torch.clamp(g[0] / p.n_vis, min=0.0)
        else:
            out["gradient"] = g[0] if one else g
    return out
