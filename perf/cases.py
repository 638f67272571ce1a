"""Timed cases of the framework: what a program that uses it has it do, through
its public entry points, from the smallest calls to the largest.

Kinds of case:
  poisson   a batch of standalone isolated solves on device grids
  step      integration cycles of one context, then the state read back
  forces    one field solve with accelerations and potentials on the host
  batch     uneven contexts stepped together, then their states read back
  segment   loss and gradients of a differentiable segment (torch.autograd)
  disc      the disc diagnostics and Fourier modes of a snapshot

FP32 contexts take FP32-representable inputs, and their states are returned
as FP32 tensors (which hold them exactly).  Their runs are short: a cell is
decided by rounding, so a particle whose position differs in the last bit can
read another cell's stencil, and over many steps two runs of the same FP32
program drift apart.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1210_1736_amd import autograd, sbx

DISC, BULGE, HALO, SAT = 0, 1, 2, 3
DT = 0.0025  # a fraction of the time a particle takes to cross an inner cell


def listed():
    return [
        # one small grid: a caller's inner loop, bound by launches
        {"name": "poisson_16_fp32", "kind": "poisson", "prec": 32, "n": 16, "batch": 1, "q": 1.0},
        # a few flattened middle grids in FP64, the precision the fields are validated in
        {"name": "poisson_64_fp64", "kind": "poisson", "prec": 64, "n": 64, "batch": 6, "q": 0.5},
        # the five grids of a galaxy: the solves/s figure
        {"name": "poisson_128_fp32", "kind": "poisson", "prec": 32, "n": 128, "batch": 5, "q": 0.25},
        # the largest grids (the ensemble's and the segment's)
        {"name": "poisson_256_fp32", "kind": "poisson", "prec": 32, "n": 256, "batch": 3, "q": 1.0},
        # a small three-level model stepped interactively: launches count
        {"name": "step_small_32_fp32", "kind": "step", "prec": 32, "n": 32, "levels": 3, "parts": 20011,
         "gals": 1, "centring": "com", "fixed": False, "steps": 5, "diag": 0},
        # the isolated Plummer cube of side 10a
        {"name": "step_plummer_64_fp64", "kind": "step", "prec": 64, "n": 64, "levels": 1, "parts": 100000,
         "gals": 1, "centring": "fixed", "fixed": False, "steps": 10, "diag": 0},
        # the disc-bulge-halo galaxy of the benchmark with its states handed on (to a display or an
        # analysis), a record of the diagnostics every 10 steps
        {"name": "step_galaxy_128_fp32", "kind": "step", "prec": 32, "n": 128, "levels": 3, "parts": 8500000,
         "gals": 1, "centring": "com", "fixed": False, "steps": 4, "diag": 10},
        # a galaxy and its satellite followed by their density maxima, merged global grid, the
        # reproducible mass assignment
        {"name": "step_satellite_64_fp64", "kind": "step", "prec": 64, "n": 64, "levels": 3, "parts": 1000003,
         "gals": 2, "centring": "density", "fixed": True, "steps": 10, "diag": 0},
        # accelerations and potentials of a model's particles on the host
        {"name": "forces_128_fp64", "kind": "forces", "prec": 64, "n": 128, "levels": 3, "parts": 300007,
         "gals": 1, "centring": "com"},
        # sinking-satellite runs of uneven size sharing the GPU
        {"name": "batch_uneven_fp32", "kind": "batch", "prec": 32, "grids": "64,64,128,128,128,256",
         "parts": "100003,1200000,180001,600000,1999999,400009", "steps": 2},
        # gradients for the largest single grid, six cycles
        {"name": "segment_256_fp32", "kind": "segment", "prec": 32, "n": 256, "levels": 1, "parts": 2050000,
         "steps": 6, "ckpt": 2},
        # one snapshot of the benchmark galaxy analysed (2M disc particles)
        {"name": "disc_snapshot_fp32", "kind": "disc", "prec": 32, "parts": 8500000, "bins": 100,
         "modes": 4},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["poisson", "poisson", "poisson", "step", "step", "step", "forces", "batch",
                       "segment", "disc"])
    prec = rng.choice([32, 64])
    if kind == "poisson":
        n = rng.choice([8, 16, 32, 64, 128, 256])
        most = min(64, (3 * 256 ** 3 * 32) // (n ** 3 * prec))
        return {"kind": kind, "prec": prec, "n": n, "batch": _log(rng, 1, most),
                "q": rng.choice([1.0, 0.5, 0.25])}
    if kind in ("step", "forces"):
        levels = rng.choice([1, 3, 3])
        n = rng.choice([32, 64, 128]) if levels == 3 else rng.choice([16, 32, 64, 128])
        gals = rng.choice([1, 1, 2]) if levels == 3 else 1
        c = {"kind": kind, "prec": prec, "n": n, "levels": levels, "gals": gals,
             "parts": _log(rng, 5000, 4000000 if kind == "step" else 1000000),
             "centring": rng.choice(["com", "com", "density", "fixed"]) if levels == 3 else "fixed"}
        if kind == "step":
            c |= {"fixed": rng.random() < 0.25, "steps": rng.randint(1, 4 if prec == 32 else 6),
                  "diag": rng.choice([0, 0, 3])}
        return c
    if kind == "batch":
        k = rng.randint(2, 6)
        grids = [rng.choice([64, 128]) for _ in range(k)]
        return {"kind": kind, "prec": 32, "grids": ",".join(map(str, grids)),
                "parts": ",".join(str(_log(rng, 100000, 2000000)) for _ in range(k)),
                "steps": rng.randint(1, 3)}
    if kind == "segment":
        steps = rng.randint(2, 6)
        return {"kind": kind, "prec": prec, "n": rng.choice([32, 64, 128]), "levels": rng.choice([1, 3]),
                "parts": _log(rng, 10000, 1000000), "steps": steps, "ckpt": rng.randint(1, min(4, steps))}
    return {"kind": kind, "prec": prec, "parts": _log(rng, 20000, 8000000), "bins": _log(rng, 10, 200),
            "modes": rng.randint(0, 8)}


# ------------------------------------------------------------------ models --
def _radii(g, n, r, cdf):
    """Radii by the inverse of a tabulated cumulative mass."""
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * cdf[-1]
    k = torch.searchsorted(cdf, u).clamp(1, cdf.numel() - 1)
    t = (u - cdf[k - 1]) / (cdf[k] - cdf[k - 1])
    return r[k - 1] + t * (r[k] - r[k - 1])


def _dirs(g, n):
    z = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    p = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (2 * math.pi)
    s = torch.sqrt(1 - z * z)
    return torch.stack([s * torch.cos(p), s * torch.sin(p), z], 1)


def _normal(g, *shape):
    return torch.randn(*shape, generator=g, device="cuda", dtype=torch.float64)


M_DISC, M_BULGE, M_HALO = 1.0, 2.14 / 4.82, 20.0 / 4.82


def _disc_cdf(r):
    return 1 - (1 + r) * torch.exp(-r)


def _bulge_cdf(r):
    return (r / (r + 0.2)) ** 2


def _halo_cdf(r):
    return torch.log1p(r / 6.72) - (r / 6.72) / (1 + r / 6.72)


def _circular(r):
    """Circular speed of the whole galaxy (spherical approximation)."""
    t = lambda v: torch.tensor(v, device="cuda", dtype=torch.float64)
    m = (M_DISC * _disc_cdf(r.clamp(max=10.0)) / _disc_cdf(t(10.0))
         + M_BULGE * _bulge_cdf(r.clamp(max=2.8)) / _bulge_cdf(t(2.8))
         + M_HALO * _halo_cdf(r.clamp(max=18.0)) / _halo_cdf(t(18.0)))
    return torch.sqrt(m / r.clamp(min=1e-6))


def _galaxy(g, n):
    """Exponential sech^2 disc, Hernquist bulge and NFW-like halo with the
    benchmark galaxy's shares of particles (2 : 0.5 : 6) and masses; the
    central cusps smoothed over a few cells, as a model relaxed on the grids
    has them."""
    nd, nb = max(1, n * 4 // 17), max(1, n // 17)
    nh = n - nd - nb
    rg = lambda hi: torch.cat([torch.zeros(1, device="cuda", dtype=torch.float64),
                               torch.logspace(-5, math.log10(hi), 4000, device="cuda", dtype=torch.float64)])
    r = rg(10.0)
    R = _radii(g, nd, r, _disc_cdf(r))
    p = torch.rand(nd, generator=g, device="cuda", dtype=torch.float64) * (2 * math.pi)
    u = torch.rand(nd, generator=g, device="cuda", dtype=torch.float64) * 2 - 1
    c, s = torch.cos(p), torch.sin(p)
    xd = torch.stack([R * c, R * s, 0.1 * torch.atanh(u * math.tanh(10.0))], 1)
    vc, sig = _circular(R), 0.35 * torch.exp(-R / 2)
    k = _normal(g, nd, 3)
    vr, vp = sig * k[:, 0], vc + 0.7 * sig * k[:, 1]
    vd = torch.stack([vr * c - vp * s, vr * s + vp * c, 0.5 * sig * k[:, 2]], 1)

    def ball(n, cdf, hi):
        r = rg(hi)
        rr = _radii(g, n, r, cdf(r))
        v = _normal(g, n, 3).clamp(-2.5, 2.5) * (0.6 * _circular(rr))[:, None]
        return rr[:, None] * _dirs(g, n) + 0.06 * _normal(g, n, 3), v

    xb, vb = ball(nb, _bulge_cdf, 2.8)
    xh, vh = ball(nh, _halo_cdf, 18.0)
    m = torch.cat([torch.full((k,), M / k, device="cuda", dtype=torch.float64)
                   for k, M in ((nd, M_DISC), (nb, M_BULGE), (nh, M_HALO))])
    comp = torch.cat([torch.full((k,), i, device="cuda", dtype=torch.int8)
                      for k, i in ((nd, DISC), (nb, BULGE), (nh, HALO))])
    return torch.cat([xd, xb, xh]), torch.cat([vd, vb, vh]), m, comp


def _plummer(g, n, M, a, cut):
    u = torch.rand(n, generator=g, device="cuda", dtype=torch.float64) * (cut ** 3 / (cut ** 2 + a ** 2) ** 1.5)
    r = a / torch.sqrt(u.clamp(min=1e-30) ** (-2 / 3) - 1)
    sig = torch.sqrt(M / (6 * torch.sqrt(r * r + a * a)))
    return r[:, None] * _dirs(g, n), _normal(g, n, 3).clamp(-2.5, 2.5) * sig[:, None]


def _flat(n):
    """Smallest flattening of 1/4, 1/2, 1 that the radii 1, 4, 20 admit."""
    need = max(0.25, 20 / (n - 4))
    return next(q for q in (0.25, 0.5, 1.0) if q >= need)


def _model(c, seed, n_grid, parts):
    """(x, v, m, comp, gal), hierarchies [(levels, centre)] of a case."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 60))
    if c.get("levels") == 1:
        if c["kind"] == "segment":  # disc, halo and a satellite on one fixed grid
            ns = max(1, parts // 41)
            x, v, m, comp = _galaxy(g, parts - ns)
            r = x.norm(dim=1, keepdim=True)
            x = x * (10.5 / torch.clamp(r, min=10.5))  # the halo cut to the grid
            ps, vs = _plummer(g, ns, 0.1, 0.6, 2.0)
            x = torch.cat([x, ps + torch.tensor([8.0, 0, 0], device="cuda", dtype=torch.float64)])
            v = torch.cat([v, vs + torch.tensor([0, 0.8, 0], device="cuda", dtype=torch.float64)])
            m = torch.cat([m, torch.full((ns,), 0.1 / ns, device="cuda", dtype=torch.float64)])
            comp = torch.cat([comp, torch.full((ns,), SAT, device="cuda", dtype=torch.int8)])
            hier = [([(n_grid, 12.0, 1.0)], (0.0, 0.0, 0.0))]
        else:
            x, v = _plummer(g, parts, 1.0, 1.0, 4.5)
            m = torch.full((parts,), 1.0 / parts, device="cuda", dtype=torch.float64)
            comp = torch.full((parts,), SAT, device="cuda", dtype=torch.int8)
            hier = [([(n_grid, 5.0, 1.0)], (0.0, 0.0, 0.0))]
        gal = torch.zeros(parts, device="cuda", dtype=torch.int8)
    else:
        q = _flat(n_grid)
        hier = [([(n_grid, 1.0, q), (n_grid, 4.0, q), (n_grid, 20.0, 1.0)], (0.0, 0.0, 0.0))]
        ns = max(1, parts // 43) if c.get("gals", 1) == 2 else 0
        x, v, m, comp = _galaxy(g, parts - ns)
        gal = torch.zeros(parts, device="cuda", dtype=torch.int8)
        if ns:
            ps, vs = _plummer(g, ns, 0.1, 0.6, 3.6)
            x = torch.cat([x, ps + torch.tensor([10.0, 0, 0], device="cuda", dtype=torch.float64)])
            v = torch.cat([v, vs + torch.tensor([0, 0.55, 0.1], device="cuda", dtype=torch.float64)])
            m = torch.cat([m, torch.full((ns,), 0.1 / ns, device="cuda", dtype=torch.float64)])
            comp = torch.cat([comp, torch.full((ns,), SAT, device="cuda", dtype=torch.int8)])
            gal[-ns:] = 1
            hier.append(([(n_grid, 1.0, 1.0), (n_grid, 6.0, 1.0), (n_grid, 20.0, 1.0)], (10.0, 0.0, 0.0)))
    if c["prec"] == 32:
        x, v, m = (t.float().double() for t in (x, v, m))
    return (x.contiguous(), v.contiguous(), m, comp, gal), hier


_CENTRING = {"fixed": sbx.SBX_CENTRE_FIXED, "com": sbx.SBX_CENTRE_COM, "density": sbx.SBX_CENTRE_DENSITY}


def _context(c, seed, n_grid, parts, centring, merge):
    (x, v, m, comp, gal), hier = _model(c, seed, n_grid, parts)
    ctx = sbx.Context(prec=sbx.SBX_FP64 if c["prec"] == 64 else sbx.SBX_FP32)
    if merge:
        ctx.sbx_set_outer_merge(1)
    ctx.sbx_build_grids([sbx.make_hierarchy(lv, _CENTRING[centring], cen) for lv, cen in hier])
    if c.get("fixed"):
        ctx.sbx_set_deterministic_deposit(1)
    torch.cuda.synchronize()
    ctx.sbx_load_particles_device(parts, x.data_ptr(), v.data_ptr(), m.data_ptr(), comp.data_ptr(),
                                  gal.data_ptr())
    return ctx


def _readback(parts):
    return {"x": torch.empty((parts, 3), device="cuda", dtype=torch.float64),
            "v": torch.empty((parts, 3), device="cuda", dtype=torch.float64),
            "lost": torch.empty(parts, device="cuda", dtype=torch.uint8)}


def _state_of(ctx, b, prec):
    ctx.sbx_get_particles_device(b["x"].data_ptr(), b["v"].data_ptr(), b["lost"].data_ptr())
    t = torch.float64 if prec == 64 else torch.float32
    return {"x": b["x"].to(t), "v": b["v"].to(t), "lost": b["lost"]}


def _instances(c):
    return list(zip(map(int, c["grids"].split(",")), map(int, c["parts"].split(","))))


DISC_QUERY = {"annulus": (3.0, 3.4), "n_z": 40, "z_max": 1.0}
MODE_BINS, MODE_RMAX = 64, 8.0


# ------------------------------------------------------------- the contract --
def prepare(case, seed):
    c = case
    s = {"case": c}
    if c["kind"] == "poisson":
        s["rho"] = _density(c, seed)
        s["phi"] = torch.empty_like(s["rho"])
        s["plan"] = sbx.Poisson(c["n"], 4.0, c["q"], prec=sbx.SBX_FP64 if c["prec"] == 64 else sbx.SBX_FP32,
                                stream=torch.cuda.current_stream().cuda_stream)
    elif c["kind"] == "step":
        s["ctx"] = _context(c, seed, c["n"], c["parts"], c["centring"], c["gals"] == 2)
        s["out"] = _readback(c["parts"])
    elif c["kind"] == "forces":
        s["ctx"] = _context(c, seed, c["n"], c["parts"], c["centring"], False)
    elif c["kind"] == "batch":
        s["ctxs"] = [_context(dict(c, levels=3, gals=2), seed * 64 + k, n, parts, "com", False)
                     for k, (n, parts) in enumerate(_instances(c))]
        s["batch"] = sbx.Batch(s["ctxs"])
        s["out"] = [_readback(parts) for _, parts in _instances(c)]
    elif c["kind"] == "segment":
        (x, v, m, comp, gal), hier = _model(c, seed, c["n"], c["parts"])
        t = torch.float64 if c["prec"] == 64 else torch.float32
        s["xvm"] = [a.to(t).requires_grad_(True) for a in (x, v, m)]
        s["comp"], s["gal"] = comp.cpu().numpy(), gal.cpu().numpy()
        s["ctx"] = sbx.Context(prec=sbx.SBX_FP64 if c["prec"] == 64 else sbx.SBX_FP32)
        s["ctx"].sbx_build_grids([sbx.make_hierarchy(lv, sbx.SBX_CENTRE_FIXED, cen) for lv, cen in hier])
    else:
        # a snapshot of a run: fixed centres, and a step of no length leaves
        # the particles where they are in the library's own order
        s["ctx"] = _context(c, seed, 64, c["parts"], "fixed", False)
        s["ctx"].sbx_step(0.0, 1)
        s["ctx"].sbx_sync()
    return s


def run(state):
    c = state["case"]
    if c["kind"] == "poisson":
        state["plan"].sbx_poisson_solve(c["batch"], state["rho"].data_ptr(), state["phi"].data_ptr())
        return state["phi"]
    if c["kind"] == "step":
        state["ctx"].sbx_step(DT, c["steps"], c["diag"])
        return _state_of(state["ctx"], state["out"], c["prec"])
    if c["kind"] == "forces":
        acc, pot = state["ctx"].sbx_compute_forces()
        if c["prec"] == 32:
            acc, pot = acc.astype(np.float32), pot.astype(np.float32)
        return {"acc": acc, "pot": pot}
    if c["kind"] == "batch":
        state["batch"].sbx_batch_step(DT, c["steps"])
        state["batch"].sbx_batch_sync()
        return [_state_of(ctx, b, c["prec"]) for ctx, b in zip(state["ctxs"], state["out"])]
    if c["kind"] == "segment":
        x, v, m = state["xvm"]
        loss = autograd.segment_loss(state["ctx"], x, v, m, state["comp"], state["gal"], DT, c["steps"],
                                     c["ckpt"], DISC, 0)
        gx, gv, gm = torch.autograd.grad(loss, (x, v, m))
        return {"loss": loss.detach().to(x.dtype), "gx": gx, "gv": gv, "gm": gm}
    d = state["ctx"].sbx_disc_analysis(c["bins"], **DISC_QUERY)
    d["modes"] = state["ctx"].sbx_disc_modes(MODE_BINS, MODE_RMAX, c["modes"])
    return d


def _solve_work(n, esz):
    """Bytes and operations of one isolated solve: the grid in and out and the
    transformed Green's function; the transforms of the padded lines that
    are not all zero."""
    L = 2 * n
    lines = 0.5 * n * n + n * (n + 1) + L * (n + 1)
    return 2 * n ** 3 * esz + (n + 1) ** 3 * esz, 2 * lines * 5 * L * math.log2(L)


def _step_work(n, parts, levels, gals, esz, merge=False):
    """One cycle: each particle's position, velocity and mass in, position and
    velocity out; its cells, stencils and kick; the solves."""
    solves = (5 * gals - (gals - 1 if merge else 0)) if levels == 3 else 1
    b, f = _solve_work(n, esz)
    return parts * 13 * esz + solves * b, parts * gals * 300 + solves * f


def work(case):
    c = case
    esz = c["prec"] // 8
    if c["kind"] == "poisson":
        b, f = _solve_work(c["n"], esz)
        h = (c["n"] + 1) ** 3 * esz
        b, f = c["batch"] * (b - h) + h, c["batch"] * f
    elif c["kind"] == "step":
        b, f = (c["steps"] * w for w in _step_work(c["n"], c["parts"], c["levels"], c["gals"], esz,
                                                   c["gals"] == 2))
        b += c["parts"] * (6 * esz + 1)
    elif c["kind"] == "forces":
        b, f = _step_work(c["n"], c["parts"], c["levels"], c["gals"], esz)
        b += c["parts"] * 4 * 8
    elif c["kind"] == "batch":
        ws = [_step_work(n, p, 3, 2, esz) for n, p in _instances(c)]
        b, f = (c["steps"] * sum(w[k] for w in ws) for k in (0, 1))
        b += sum(p for _, p in _instances(c)) * (6 * esz + 1)
    elif c["kind"] == "segment":
        # the cycles once forwards and once backwards (adjoint solves)
        b, f = (2 * c["steps"] * w for w in _step_work(c["n"], c["parts"], c["levels"], 1, esz))
        b += c["parts"] * 7 * 8
    else:
        b, f = c["parts"] * (7 * esz + 3), c["parts"] * 60
    return {"bytes": float(b), "flops": float(f)}


# -------------------------------------------------- the method in 64 bits ---
# Plain torch, float64 on the GPU: cells by rounding to the nearest grid
# point, convolution with 1/r on the doubled grid, the central differences
# with their second-order Taylor terms, leapfrog.  Cells are held constant in
# derivatives.
def _density(c, seed):
    """Cell masses with a galaxy's contrast: empty to crowded cells."""
    g = torch.Generator(device="cuda").manual_seed(int(seed) % (1 << 60))
    t = torch.float64 if c["prec"] == 64 else torch.float32
    shape = (c["batch"], c["n"], c["n"], c["n"])
    a = torch.linspace(-1, 1, c["n"], device="cuda", dtype=t)
    r2 = a[:, None, None] ** 2 + a[None, :, None] ** 2 + a[None, None, :] ** 2
    u = torch.rand(shape, generator=g, device="cuda", dtype=t)
    return u * u / (r2 + 0.01)


class _Level:
    def __init__(self, n, R, q):
        self.n, self.R, self.q = n, R, q
        self.l = 2 * R / (n - 4)
        self.d = [self.l, self.l, q * self.l]

    def cells(self, dx):
        """Nearest cells of offsets dx (particles, 3) from the grid's centre."""
        k = [torch.floor(dx[:, i] * (1.0 / self.d[i]) + self.n / 2 + 0.5) for i in range(3)]
        return torch.stack(k, 1).clamp(-2 ** 30, 2 ** 30).to(torch.int64)

    def usable(self, k):
        return ((k >= 2) & (k <= self.n - 3)).all(1)

    def inside(self, dx):
        return dx[:, 0] ** 2 + dx[:, 1] ** 2 + (dx[:, 2] * (1 / self.q)) ** 2 < self.R ** 2

    def flat(self, k):
        return (k[:, 2] * self.n + k[:, 1]) * self.n + k[:, 0]


def _greens(lv):
    L = 2 * lv.n
    k = torch.arange(L, device="cuda", dtype=torch.float64)
    k = torch.minimum(k, L - k)
    r = torch.sqrt((k * lv.d[2])[:, None, None] ** 2 + (k * lv.l)[None, :, None] ** 2
                   + (k * lv.l)[None, None, :] ** 2)
    r[0, 0, 0] = lv.l
    return torch.fft.rfftn(1 / r).real


def _solve(rho, H):
    n = rho.shape[-1]
    return torch.fft.irfftn(torch.fft.rfftn(rho, s=(2 * n,) * 3) * H, s=(2 * n,) * 3)[:n, :n, :n]


def _field(F, lv, k, dx):
    """Acceleration and potential of field F at offsets dx in cells k."""
    n = lv.n
    F, at = F.reshape(-1), lv.flat(k)
    p = lambda x, y, z: F[at + (z * n + y) * n + x]
    D = [dx[:, i] - (k[:, i].to(torch.float64) - n / 2) * lv.d[i] for i in range(3)]
    e = [(1, 0, 0), (0, 1, 0), (0, 0, 1)]
    c = p(0, 0, 0)
    up = [p(*a) for a in e]
    dn = [p(*(-i for i in a)) for a in e]
    grad = [(up[i] - dn[i]) / (2 * lv.d[i]) for i in range(3)]
    h = [[None] * 3 for _ in range(3)]
    for i in range(3):
        h[i][i] = (up[i] + dn[i] - 2 * c) / lv.d[i] ** 2
        for j in range(i):
            s = lambda a, b: p(*(a * e[i][w] + b * e[j][w] for w in range(3)))
            h[i][j] = h[j][i] = (s(1, 1) - s(1, -1) - s(-1, 1) + s(-1, -1)) / (4 * lv.d[i] * lv.d[j])
    acc = torch.stack([grad[i] + sum(h[i][j] * D[j] for j in range(3)) for i in range(3)], 1)
    pot = c + sum(grad[i] * D[i] for i in range(3)) + 0.5 * sum(h[i][j] * D[i] * D[j]
                                                              for i in range(3) for j in range(3))
    return acc, pot


class _System:
    """The nested-grid particle-mesh model of a set of hierarchies."""

    def __init__(self, hier, centring):
        self.gal = [[_Level(*lv) for lv in levels] for levels, _ in hier]
        self.centring = centring
        self.centre = [torch.tensor(cen, device="cuda", dtype=torch.float64) for _, cen in hier]
        self.H = {}

    def solve(self, rho, lv):
        key = (lv.n, lv.R, lv.q)
        if key not in self.H:
            self.H[key] = _greens(lv)
        return _solve(rho, self.H[key])

    def lost(self, x):
        top = self.gal[0][-1]
        return ~top.usable(top.cells(x))

    def move_centres(self, x, m, gal, live):
        if self.centring == "fixed":
            return
        for g, levels in enumerate(self.gal):
            own = live & (gal == g)
            if self.centring == "density":
                lv = levels[0]
                k = lv.cells(x - self.centre[g])
                on = own & ((k >= 0) & (k < lv.n)).all(1)
                if not bool(on.any()):
                    continue
                shift = 62 - math.frexp(float(m.max()))[1] - x.shape[0].bit_length()
                w = torch.floor(m * 2.0 ** shift).to(torch.int64)
                hist = torch.zeros(lv.n ** 3, device="cuda", dtype=torch.int64)
                hist.index_add_(0, lv.flat(k)[on], w[on])
                best = int((hist == hist.max()).nonzero()[0, 0])
                b = torch.tensor([best % lv.n, best // lv.n % lv.n, best // lv.n ** 2], device="cuda")
                own = own & ((k - b).abs() <= 1).all(1)
            M = m[own].sum()
            if float(M) > 0:
                self.centre[g] = (m[own, None] * x[own]).sum(0) / M

    def forces(self, x, m, gal, live):
        """Accelerations and potentials (zero where not live)."""
        self.move_centres(x.detach(), m.detach(), gal, live)
        acc, pot = torch.zeros_like(x), torch.zeros_like(m)
        for g, levels in enumerate(self.gal):
            cen = self.centre[g]
            dx, ox = x - cen, x
            if len(levels) == 1:
                dx = ox = x - cen
            k = [lv.cells((ox if i == len(levels) - 1 else dx).detach()) for i, lv in enumerate(levels)]
            ok = [lv.usable(a) for lv, a in zip(levels, k)]
            top = len(levels) - 1
            if top:
                core = live & ok[0] & ok[1] & ok[2] & levels[0].inside(dx.detach())
                ring = live & ok[1] & ok[2] & levels[1].inside(dx.detach()) & ~core
                outer = live & ok[2] & ~core & ~ring
                parts = [(core, 0), (ring, 1), (core, 1), (outer, 2), (core | ring, 2)]
            else:
                outer = live & ok[0]
                parts = [(outer, 0)]
            phi = []
            for who, i in parts:  # grids 1, 3, 2, 5, 4
                lv, w = levels[i], (who & (gal == g)).nonzero()[:, 0]
                rho = torch.zeros(lv.n ** 3, device="cuda", dtype=torch.float64)
                rho = rho.index_add(0, lv.flat(k[i][w]), m[w])
                phi.append(self.solve(rho.view(lv.n, lv.n, lv.n), lv))
            if top:
                reads = [(core, [(phi[0], 0), (phi[1], 1), (phi[3], 2)]),
                         (ring, [(phi[1] + phi[2], 1), (phi[3], 2)]), (outer, [(phi[3] + phi[4], 2)])]
            else:
                reads = [(outer, [(phi[0], 0)])]
            for who, fields in reads:
                w = who.nonzero()[:, 0]
                for F, i in fields:
                    a, p = _field(F, levels[i], k[i][w], (ox if i == top else dx)[w])
                    acc = acc.index_add(0, w, a)
                    pot = pot.index_add(0, w, -p)
        return acc, pot

    def steps(self, x, v, m, gal, count):
        gone = torch.zeros(x.shape[0], device="cuda", dtype=torch.bool)
        for _ in range(count):
            gone = gone | self.lost(x.detach())
            live = ~gone
            acc, _ = self.forces(x, m, gal, live)
            v = torch.where(live[:, None], v + DT * acc, v)
            x = torch.where(live[:, None], x + DT * v, x)
            gone = gone | (live & self.lost(x.detach()))
        return x, v, gone


def _exact_disc(x, v, m, comp, c):
    s = comp == DISC
    x, v, m = x[s], v[s], m[s]
    bulk = (m[:, None] * v).sum(0) / m.sum()
    u = v - bulk
    R = torch.sqrt(x[:, 0] ** 2 + x[:, 1] ** 2)
    vR = (x[:, 0] * u[:, 0] + x[:, 1] * u[:, 1]) / R
    vp = (x[:, 0] * u[:, 1] - x[:, 1] * u[:, 0]) / R
    order = torch.sort(R, stable=True)[1]
    n, nb = R.numel(), c["bins"]
    count = torch.tensor([n // nb + (1 if k < n % nb else 0) for k in range(nb)], device="cuda")
    at = torch.repeat_interleave(torch.arange(nb, device="cuda"), count)
    mean = lambda q: torch.zeros(nb, device="cuda", dtype=torch.float64).index_add(0, at, q[order]) / count
    br, bv, bz = mean(R), mean(vp), torch.sqrt(mean(x[:, 2] ** 2))
    k = torch.searchsorted(br, R, right=True).clamp(1, max(1, nb - 1))
    if nb > 1:
        t = ((R - br[k - 1]) / (br[k] - br[k - 1])).clamp(0, 1)
        vc = bv[k - 1] + t * (bv[k] - bv[k - 1])
    else:
        vc = bv[0].expand(n)
    heat = (0.5 * m * (vR ** 2 + (vp - vc) ** 2 + u[:, 2] ** 2)).sum()
    (lo, hi), nz, zm = DISC_QUERY["annulus"], DISC_QUERY["n_z"], DISC_QUERY["z_max"]
    a = (R >= lo) & (R < hi)
    sd = lambda q: torch.sqrt((q[a] ** 2).mean() - q[a].mean() ** 2)
    dz = 2 * zm / nz
    z = x[a, 2]
    zin = (z >= -zm) & (z < zm)
    rho = torch.zeros(nz, device="cuda", dtype=torch.float64)
    rho.index_add_(0, torch.floor((z[zin] + zm) / dz).long().clamp(max=nz - 1), m[a][zin])
    rho /= math.pi * (hi * hi - lo * lo) * dz
    dR = MODE_RMAX / MODE_BINS
    edge = torch.arange(MODE_BINS + 1, device="cuda", dtype=torch.float64) * dR
    b = torch.searchsorted(edge, R, right=True) - 1
    on = b < MODE_BINS
    area = math.pi * (edge[1:] ** 2 - edge[:-1] ** 2)
    ph = torch.atan2(x[:, 1], x[:, 0])
    modes = torch.zeros((MODE_BINS, c["modes"] + 1), device="cuda", dtype=torch.complex128)
    for q in range(c["modes"] + 1):
        w = torch.complex(m * torch.cos(q * ph), -m * torch.sin(q * ph))
        for part in ("real", "imag"):
            s = torch.zeros(MODE_BINS, device="cuda", dtype=torch.float64)
            getattr(modes, part)[:, q] = s.index_add(0, b[on], getattr(w, part)[on]) / area
    f = lambda t: float(t)
    some = int(a.sum()) > 0
    sig = [f(sd(q)) if some else 0.0 for q in (vR, vp, u[:, 2])]
    return {"e_heat": f(heat), "sig_R": sig[0], "sig_phi": sig[1], "sig_z": sig[2],
            "sig_tot2": sum(q * q for q in sig), "bulk_v": bulk.cpu().numpy(), "n_disc": n,
            "n_annulus": int(a.sum()), "bin_r": br.cpu().numpy(), "bin_vc": bv.cpu().numpy(),
            "bin_rms_z": bz.cpu().numpy(), "rho_z": rho.cpu().numpy(), "modes": modes.cpu().numpy()}


def exact(case, seed):
    c = case
    if c["kind"] == "poisson":
        lv = _Level(c["n"], 4.0, c["q"])
        H = _greens(lv)
        return torch.stack([_solve(r.double(), H) for r in _density(c, seed)])
    if c["kind"] == "batch":
        out = []
        for k, (n, parts) in enumerate(_instances(c)):
            (x, v, m, _, gal), hier = _model(dict(c, levels=3, gals=2), seed * 64 + k, n, parts)
            x, v, gone = _System(hier, "com").steps(x, v, m, gal, c["steps"])
            out.append({"x": x, "v": v, "lost": gone.to(torch.uint8)})
        return out
    (x, v, m, comp, gal), hier = _model(c, seed, c.get("n", 64), c["parts"])
    if c["kind"] == "step":
        x, v, gone = _System(hier, c["centring"]).steps(x, v, m, gal, c["steps"])
        return {"x": x, "v": v, "lost": gone.to(torch.uint8)}
    if c["kind"] == "forces":
        s = _System(hier, c["centring"])
        acc, pot = s.forces(x, m, gal, ~s.lost(x))
        return {"acc": acc, "pot": pot}
    if c["kind"] == "segment":
        x, v, m = (t.requires_grad_(True) for t in (x, v, m))
        _, vz, gone = _System(hier, "fixed").steps(x, v, m, gal, c["steps"])
        sel = (comp == DISC) & (gal == 0) & ~gone
        loss = (0.5 * m[sel] * vz[sel, 2] ** 2).sum()
        gx, gv, gm = torch.autograd.grad(loss, (x, v, m))
        return {"loss": loss.detach(), "gx": gx, "gv": gv, "gm": gm}
    return _exact_disc(x, v, m, comp, c)
