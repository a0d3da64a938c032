"""Timed cases of the solver: what its users run, over the sizes they run it at.

A case names a workload (``kind``), its sizes, the stored precision and how
many steps one pass takes.  ``prepare`` makes the initial data from the seed
and sets up the grid or batch, ``run`` is one pass through the public entry
points and returns the advanced conserved densities, ``exact`` is the same
pass in plain FP64 torch, written from the scheme's formulas.
"""
import math
import random
from types import SimpleNamespace

import numpy as np
import torch

from paper_1607_01105_amd.ppml import Batch, Grid

GH = 3  # ghost layers of the scheme


def listed():
    return [
        # one small shock tube, stepped in the calls of 64 that run_to makes
        {"name": "riemann_1d_512_fp64", "kind": "riemann", "nx": 512, "prec": "fp64", "steps": 64},
        # Kelvin-Helmholtz at the paper's mesh: a 2-D grid of one tile per CU
        {"name": "shear_2d_256_fp32", "kind": "shear", "nx": 256, "ny": 256, "prec": "fp32", "steps": 32},
        # Rayleigh-Taylor at the paper's mesh (ragged, walls, uniform gravity),
        # in calls shorter than the captured chunk
        {"name": "layers_2d_100x600_fp64", "kind": "layers", "nx": 100, "ny": 600, "prec": "fp64", "steps": 20},
        # the Sedov mesh: too few tiles to fill the chip
        {"name": "box_3d_100_fp32", "kind": "box", "nx": 100, "ny": 100, "nz": 100, "prec": "fp32", "steps": 10},
        # the headline benchmark's box
        {"name": "box_3d_256_fp32", "kind": "box", "nx": 256, "ny": 256, "nz": 256, "prec": "fp32", "steps": 2},
        # odd sizes, walls on one axis, FP64
        {"name": "box_3d_131x97x75_fp64", "kind": "box", "nx": 131, "ny": 97, "nz": 75, "prec": "fp64", "steps": 4,
         "bc": "mixed"},
        # rotating disk in a logarithmic potential, outflow faces, FP64
        {"name": "disk_3d_512x512x64_fp64", "kind": "disk", "nx": 512, "ny": 512, "nz": 64, "prec": "fp64",
         "steps": 1},
        # self-gravitating ball: a potential solve before the step
        {"name": "ball_3d_256_fp32", "kind": "ball", "nx": 256, "ny": 256, "nz": 256, "prec": "fp32", "steps": 1},
        # galactic disk: isothermal gas, halo potential and self-gravity, FP64
        {"name": "galaxy_3d_150_fp64", "kind": "galaxy", "nx": 150, "ny": 150, "nz": 150, "prec": "fp64", "steps": 1},
        # many small 1-D and 2-D grids in one graph-replayed batch
        {"name": "batch_mix_fp32", "kind": "batch", "n1d": 24, "n2d": 24, "n3d": 0, "prec": "fp32", "steps": 50},
        # a round of the server: 2-D and 3-D requests resident together
        {"name": "served_round_fp32", "kind": "batch", "n1d": 0, "n2d": 6, "n3d": 6, "prec": "fp32", "steps": 10},
        # restart: host fields to the device, FP64 totals, fields back to the host
        {"name": "checkpoint_3d_128_fp32", "kind": "checkpoint", "nx": 128, "ny": 128, "nz": 128, "prec": "fp32",
         "steps": 0},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["riemann", "blast", "shear", "layers", "box2", "box3", "box3", "disk", "ball", "ball", "galaxy",
                       "mix", "served", "checkpoint"])
    prec = rng.choice(["fp32", "fp64"])
    if kind in ("riemann", "blast"):
        return {"kind": kind, "nx": _log_int(rng, 64, 4096), "prec": prec, "steps": _log_int(rng, 8, 128)}
    if kind == "shear":
        n = _log_int(rng, 48, 512)
        return {"kind": kind, "nx": n, "ny": n, "prec": prec, "steps": _log_int(rng, 4, 64)}
    if kind == "layers":
        n = _log_int(rng, 24, 160)
        return {"kind": kind, "nx": n, "ny": 6 * n, "prec": prec, "steps": _log_int(rng, 4, 64)}
    if kind in ("box2", "box3"):
        three = kind == "box3"
        c = {"kind": "box", "nx": _log_int(rng, 24, 220 if three else 768), "ny": _log_int(rng, 24, 220 if three else 768)}
        if three:
            c["nz"] = _log_int(rng, 24, 220)
        c.update(prec=prec, steps=_log_int(rng, 1, 4 if three else 32), bc=rng.choice(["periodic", "outflow", "mixed"]))
        option = rng.choice(["", "", "first_order", "isothermal"])
        if option:
            c[option] = True
        return c
    if kind == "disk":
        n = _log_int(rng, 96, 384)
        return {"kind": kind, "nx": n, "ny": n, "nz": _log_int(rng, 16, 64), "prec": "fp64", "steps": _log_int(rng, 1, 4),
                "isothermal": rng.random() < 0.5}
    if kind == "ball":
        n = _log_int(rng, 48, 224)
        return {"kind": kind, "nx": n, "ny": n if rng.random() < 0.5 else _log_int(rng, 48, 224), "nz": n, "prec": prec,
                "steps": _log_int(rng, 1, 3)}
    if kind == "galaxy":
        n = _log_int(rng, 48, 144)
        return {"kind": kind, "nx": n, "ny": n, "nz": n, "prec": "fp64", "steps": _log_int(rng, 1, 3)}
    if kind == "mix":
        return {"kind": "batch", "n1d": rng.randint(4, 24), "n2d": rng.randint(4, 24), "n3d": 0, "prec": prec,
                "steps": _log_int(rng, 8, 50)}
    if kind == "served":
        return {"kind": "batch", "n1d": 0, "n2d": rng.randint(1, 6), "n3d": rng.randint(1, 5), "prec": "fp32",
                "steps": _log_int(rng, 2, 9)}
    nd = rng.choice([1, 2, 3])
    c = {"kind": "checkpoint", "nx": _log_int(rng, 24, 128) if nd == 3 else _log_int(rng, 64, 1024)}
    if nd >= 2:
        c["ny"] = _log_int(rng, 24, 128) if nd == 3 else _log_int(rng, 64, 1024)
    if nd == 3:
        c["nz"] = _log_int(rng, 24, 128)
    return {**c, "prec": prec, "steps": 0}


# ---- initial data ---------------------------------------------------------
def _device():
    return torch.device("cuda" if torch.cuda.is_available() else "cpu")


def _centres(p):
    x = [p.lo[a] + (torch.arange(p.n[a], dtype=torch.float64, device=_device()) + 0.5) * p.h[a] for a in range(3)]
    return x[0][None, None, :], x[1][None, :, None], x[2][:, None, None]


def _modes(p, rng, amp=0.1):
    """1 + amp times eight random periodic modes of |k| <= 4."""
    X, Y, Z = _centres(p)
    f = torch.ones(p.n[::-1], dtype=torch.float64, device=_device())
    for _ in range(8):
        k = (0, 0, 0)
        while not 1 <= sum(c * c for c in k) <= 16:
            k = tuple(rng.randint(-4, 4) if a < p.ndim else 0 for a in range(3))
        f += amp * torch.cos(2.0 * math.pi * (k[0] * X + k[1] * Y + k[2] * Z) + rng.uniform(0.0, 2.0 * math.pi))
    return f


def _noise(p, seed, rms):
    g = torch.Generator(device=_device())
    g.manual_seed(seed)
    return torch.exp(rms * torch.randn(p.n[::-1], dtype=torch.float64, device=_device(), generator=g))


def _describe(n, lo, hi, gamma, cfl, bc):
    ndim = len(n)
    n = tuple(n) + (1,) * (3 - ndim)
    lo = tuple(lo) + (-0.5,) * (3 - ndim)
    hi = tuple(hi) + (0.5,) * (3 - ndim)
    bc = [tuple(b) for b in bc] + [("periodic", "periodic")] * (3 - ndim)
    return SimpleNamespace(ndim=ndim, n=n, lo=lo, hi=hi, h=[(hi[a] - lo[a]) / n[a] for a in range(3)], gamma=gamma,
                           cfl=cfl, bc=bc, potential=None, isothermal=None, self_gravity=None, first_order=False)


def problem(case, seed):
    """Descriptor and primitive fields (FP64 tensors [z, y, x]) of a single grid."""
    rng = random.Random(seed)
    kind = case["kind"]
    n = tuple(case[a] for a in ("nx", "ny", "nz") if a in case)
    ndim = len(n)
    if kind in ("riemann", "blast"):
        wall = "outflow" if kind == "riemann" else "reflect"
        p = _describe(n, (0.0,), (1.0,), 1.4, 0.4, [(wall, wall)])
        x = _centres(p)[0]
        if kind == "riemann":  # seeded left and right states
            left, right = ((rng.uniform(0.1, 1.0), rng.uniform(-1.0, 1.0), rng.uniform(0.1, 1.0)) for _ in range(2))
            rho, v, pr = (torch.where(x < 0.5, a, b) for a, b in zip(left, right))
        else:  # two interacting blast waves between walls
            rho, v = torch.ones_like(x), torch.zeros_like(x)
            hot, warm = 1000.0 * rng.uniform(0.8, 1.2), 100.0 * rng.uniform(0.8, 1.2)
            pr = torch.where(x < 0.1, hot, torch.where(x < 0.9, 0.01, warm))
        p.prim = [rho.double(), v.double(), None, None, pr.double()]
    elif kind == "shear":
        p = _describe(n, (-0.5, -0.5), (0.5, 0.5), 1.4, 0.4, [("periodic", "periodic")] * 2)
        X, Y, _ = _centres(p)
        inner = (Y.abs() <= 0.25 + 0.01 * (1.0 + torch.cos(8.0 * math.pi * X + rng.uniform(0.0, 6.0)))).expand(p.n[::-1])
        one = torch.ones(p.n[::-1], dtype=torch.float64, device=_device())
        rho, vx = torch.where(inner, 2.0 * one, one), torch.where(inner, 0.5 * one, -0.5 * one)
        p.prim = [rho * _noise(p, seed, 1e-3), vx, 0.01 * (_modes(p, rng) - 1.0), None, 2.5 * one]
    elif kind == "layers":
        p = _describe(n, (-0.25, -1.5), (0.25, 1.5), 1.4, 0.2, [("periodic", "periodic"), ("reflect", "reflect")])
        X, Y, _ = _centres(p)
        one = torch.ones(p.n[::-1], dtype=torch.float64, device=_device())
        rho = torch.where(Y.abs() <= 0.75, 2.0, 1.0) * one
        above = torch.where(Y >= 0.75, 1.5 - Y, torch.where(Y >= -0.75, 2.25 - 2.0 * Y, 3.0 - Y))
        vy = 0.01 * (1.0 + torch.cos(2.0 * math.pi * Y)) * torch.cos(4.0 * math.pi * X + rng.uniform(0.0, 6.0))
        p.prim = [rho, 0.0 * one, vy * one, None, (0.15 + 0.1 * above) * one]
        p.potential = ("uniform", 0.0, 0.1, 0.0)
    elif kind in ("box", "checkpoint"):
        faces = {"outflow": [("outflow", "outflow")] * ndim,
                 "mixed": [("reflect", "outflow"), ("periodic", "periodic"), ("reflect", "reflect")][:ndim]}
        p = _describe(n, (0.0,) * ndim, (1.0,) * ndim, 5.0 / 3.0, 0.3,
                      faces.get(case.get("bc"), [("periodic", "periodic")] * ndim))
        rho = _modes(p, rng)
        d2 = sum((x - rng.uniform(0.3, 0.7)) ** 2 for x in _centres(p)[:ndim])
        if case.get("isothermal"):  # at rest pressure follows the density: start from a flow
            p.isothermal = 1.0
            v = [0.5 * (_modes(p, rng) - 1.0) if a < ndim else None for a in range(3)]
            p.prim = [rho * (1.0 + 4.0 * (d2 <= 0.01)), *v, rho * (1.0 + 4.0 * (d2 <= 0.01))]
        else:  # a hot sphere in a structured medium
            p.prim = [rho, None, None, None, torch.where(d2.expand(p.n[::-1]) <= 0.01, 100.0, 1.0).double()]
        p.first_order = bool(case.get("first_order"))
    elif kind == "disk":
        h, cs = 1.0 / n[0], 0.2
        p = _describe(n, (-0.5, -0.5, -0.5 * n[2] * h), (0.5, 0.5, 0.5 * n[2] * h), 5.0 / 3.0, 0.2,
                      [("outflow", "outflow")] * 3)
        X, Y, Z = _centres(p)
        R = torch.sqrt(X * X + Y * Y)
        H = torch.clamp(cs * torch.sqrt(R * R + 0.02 ** 2), min=2.0 * h)
        rho = torch.clamp(torch.exp(-R / 0.2) / (math.sqrt(2.0 * math.pi) * H) * torch.exp(-Z * Z / (2.0 * H * H)), min=2e-2)
        rho = rho * _noise(p, seed, 0.01)
        om = 1.0 / torch.sqrt(R * R + 0.02 ** 2)
        iso = bool(case.get("isothermal"))
        p.prim = [rho, -Y * om, X * om, None, rho * (cs * cs / (1.0 if iso else p.gamma))]
        p.potential = ("log", 1.0, 0.02, 1.0, 0.0, 0.0, 0.0)
        p.isothermal = cs if iso else None
    elif kind == "ball":  # a rotating, self-gravitating ball in a hot thin medium
        h = 4.0 / n[0]
        p = _describe(n, [-0.5 * m * h for m in n], [0.5 * m * h for m in n], 5.0 / 3.0, 0.3, [("outflow", "outflow")] * 3)
        X, Y, Z = _centres(p)
        r = torch.sqrt(X * X + Y * Y + Z * Z)
        rho = (torch.where(r <= 1.0, 2.0 * r ** 3 - 3.0 * r ** 2 + 1.0, 0.0) + 1e-2) * _noise(p, seed, 0.01)
        w = [rng.uniform(0.3, 0.6) for _ in range(3)]
        damp = torch.exp(-r * r)
        p.prim = [rho, (w[1] * Z - w[2] * Y) * damp, (w[2] * X - w[0] * Z) * damp, (w[0] * Y - w[1] * X) * damp,
                  torch.full_like(rho, 0.2)]
        p.self_gravity = 1.0
    elif kind == "galaxy":
        h, cs, r0 = 1.0 / n[0], 0.2, 0.05
        p = _describe(n, (-0.5,) * 3, (0.5,) * 3, 5.0 / 3.0, 0.2, [("outflow", "outflow")] * 3)
        X, Y, Z = _centres(p)
        R = torch.sqrt(X * X + Y * Y)
        H = torch.clamp(cs * torch.sqrt(R * R + r0 * r0), min=2.0 * h)
        rho = torch.exp(-R / 0.1) / (math.sqrt(2.0 * math.pi) * H) * torch.exp(-Z * Z / (2.0 * H * H))
        rho = torch.clamp(rho, min=2e-2) * _noise(p, seed, 1e-4)
        u = torch.clamp(R / r0, min=1e-9)
        vphi = torch.sqrt(torch.clamp(1.0 - torch.atan(u) / u, min=0.0)) / torch.clamp(R, min=1e-12)
        p.prim = [rho, -Y * vphi, X * vphi, None, rho * cs * cs]
        p.potential = ("halo", 1.0 / (4.0 * math.pi * r0 * r0), r0, r0 * 78.55 / 1.6, 0.0, 0.0, 0.0)
        p.isothermal = cs
        p.self_gravity = 1.0
    else:
        raise ValueError(kind)
    return p


def members(case, seed):
    """The grids of a batch: (case, seed) of each, sizes log-uniform as in the
    benchmark's batched mix (1-D 64-4096, 2-D sides 32-256 beside them) and
    served trace (2-D 64-512, 3-D 64-192), the same sizes for every seed."""
    size = random.Random(1000 * case["n1d"] + 100 * case["n2d"] + case["n3d"])
    out = [{"kind": "riemann", "nx": _log_int(size, 64, 4096)} for _ in range(case["n1d"])]
    if case["n3d"]:
        out += [{"kind": "box", "nx": m, "ny": m} for m in (_log_int(size, 64, 512) for _ in range(case["n2d"]))]
        out += [{"kind": "box", "nx": m, "ny": m, "nz": m} for m in (_log_int(size, 64, 192) for _ in range(case["n3d"]))]
    else:
        out += [{"kind": "box", "nx": _log_int(size, 32, 256), "ny": _log_int(size, 32, 256)} for _ in range(case["n2d"])]
    return [(c, 64 * seed + i) for i, c in enumerate(out)]


# ---- the framework's side -------------------------------------------------
def _grid(p, prec, stream=None):
    g = Grid(p.ndim, p.n[: p.ndim], p.lo, p.hi, p.gamma, p.cfl, bc=p.bc, prec=prec, potential=p.potential,
             first_order=p.first_order, self_gravity=p.self_gravity, isothermal=p.isothermal, stream=stream)
    g.set_primitive(*[None if f is None else f.expand(p.n[::-1]).contiguous().cpu().numpy() for f in p.prim])
    return g


def _fields(g):
    """The conserved densities of a grid, views of its device state."""
    u = g.state.view(torch.float64 if g.desc.prec else torch.float32)
    u = u[: (3 + g.ndim) * g.ncell].view(3 + g.ndim, *g.shape)
    return {"rho": u[0], "mom": u[1: 1 + g.ndim], "etot": u[1 + g.ndim], "eint": u[2 + g.ndim]}


def prepare(case, seed):
    s = SimpleNamespace(case=case, batch=None)
    if case["kind"] == "batch":
        s.batch = Batch(capacity=case["n1d"] + case["n2d"] + case["n3d"])
        s.grids = [_grid(problem(c, sd), case["prec"], s.batch.stream) for c, sd in members(case, seed)]
        for g in s.grids:
            s.batch.admit(g)
        return s
    p = problem(case, seed)
    s.grid = _grid(p, case["prec"])
    if case["kind"] == "checkpoint":
        s.saved = [u.cpu().numpy() for u in conserved(p)]
    return s


def run(state):
    case = state.case
    if state.batch is not None:
        state.batch.step(case["steps"], graph=True)
        return [torch.flatten(g.state.view(torch.float64 if g.desc.prec else torch.float32)) for g in state.grids]
    g = state.grid
    if case["kind"] == "checkpoint":
        g.set_conserved(state.saved, rho_mean0=1.0, t=0.5)
        return {"totals": g.totals(), "fields": g.conserved()}
    g.step(case["steps"])
    return _fields(g)


def _flops(p):
    """Floating-point operations of a step per cell: the formulas' adds,
    multiplies, divisions and square roots, shared interface values once."""
    nd, nf = p.ndim, 3 + p.ndim
    euler = 7 + nd * 113 + 4 * (1 + nd)
    lagr = nd * (12 + (0, 4, 11)[nd - 1] + nf * 37) + 46
    solve = 0
    if p.self_gravity:  # forward and inverse sine transforms, as fast ones would cost
        solve = sum(10.0 * math.log2(2 * (m + 1)) for m in p.n)
    return euler + lagr + solve


def work(case):
    w = 8 if case["prec"] == "fp64" else 4
    if case["kind"] == "batch":
        total = {"bytes": 0, "flops": 0}
        for c, _ in members(case, 0):
            one = work({**c, "prec": case["prec"], "steps": case["steps"]})
            total = {k: total[k] + one[k] for k in total}
        return total
    n = [case[a] for a in ("nx", "ny", "nz") if a in case]
    cells, nf = math.prod(n), 3 + len(n)
    if case["kind"] == "checkpoint":  # six host arrays each way, the state written once and read for totals and fields
        return {"bytes": cells * (2 * 6 * 8 + 3 * nf * w), "flops": 6 * cells}
    p = SimpleNamespace(ndim=len(n), n=n, self_gravity=case["kind"] in ("ball", "galaxy"))
    return {"bytes": 2 * nf * w * cells, "flops": case["steps"] * _flops(p) * cells}


# ---- the same pass in 64 bits ---------------------------------------------
def conserved(p):
    rho, vx, vy, vz, pr = (torch.zeros(p.n[::-1], dtype=torch.float64, device=_device()) if f is None else
                           f.expand(p.n[::-1]).contiguous() for f in p.prim)
    vy, vz = (v if a < p.ndim else 0.0 * v for a, v in ((1, vy), (2, vz)))
    e = pr / (p.gamma - 1.0)
    return [rho, rho * vx, rho * vy, rho * vz, e + 0.5 * rho * (vx * vx + vy * vy + vz * vz), e]


def _ghosted(p, u):
    """Three ghost layers per side of every active axis, filled x, then y, then z."""
    for a in range(p.ndim):
        m, (lo, hi) = p.n[a], p.bc[a]
        i = torch.arange(-GH, m + GH)
        src, flip = i.clone(), torch.zeros_like(i, dtype=torch.bool)
        for side, bc in ((i < 0, lo), (i >= m, hi)):
            if bc == "periodic":
                src = torch.where(side, i % m, src)
            elif bc == "outflow":
                src = torch.where(side, i.clamp(0, m - 1), src)
            else:
                src = torch.where(side, torch.where(i < 0, -1 - i, 2 * m - 1 - i), src)
                flip = flip | side
        src = src.to(u[0].device)
        sign = torch.where(flip, -1.0, 1.0).double().to(u[0].device).view([-1 if d == 2 - a else 1 for d in range(3)])
        u = [f.index_select(2 - a, src) for f in u]
        u[1 + a] = u[1 + a] * sign
    return u


def _cut(f, axis, start, count):
    return f.narrow(2 - axis, start, count)


def _line(p, f, a):
    """Interior on the other axes, the whole ghosted line along axis a."""
    for o in range(p.ndim):
        if o != a:
            f = _cut(f, o, GH, p.n[o])
    return f


def _parabolas(p, q, a):
    """Left and right edge values and curvature of the cells -1 .. n along a."""
    m = p.n[a] + 6
    if p.first_order:
        c = _cut(q, a, 2, m - 4)
        return c, c, torch.zeros_like(c)
    up, mid, down = _cut(q, a, 2, m - 2), _cut(q, a, 1, m - 2), _cut(q, a, 0, m - 2)
    dp, dm, dq = up - mid, mid - down, 0.5 * (up - down)
    sl = torch.minimum(dq.abs(), 2.0 * torch.minimum(dp.abs(), dm.abs()))
    sl = torch.where(dp * dm > 0, torch.copysign(sl, dq), torch.zeros_like(sl))
    face = 0.5 * (_cut(q, a, 1, m - 3) + _cut(q, a, 2, m - 3)) - (_cut(sl, a, 1, m - 3) - _cut(sl, a, 0, m - 3)) / 6.0
    c, l, r = _cut(q, a, 2, m - 4), _cut(face, a, 0, m - 4), _cut(face, a, 1, m - 4)
    flat = (r - c) * (c - l) <= 0
    d, s6 = r - l, 6.0 * (c - 0.5 * (l + r))
    left = torch.where(flat, c, torch.where(d * s6 > d * d, 3.0 * c - 2.0 * r, l))
    right = torch.where(flat, c, torch.where(d * s6 < -d * d, 3.0 * c - 2.0 * l, r))
    return left, right, 6.0 * (c - 0.5 * (left + right))


def _strips(p, par, a, z):
    """Means of the left cell's parabola next to each face and of the right cell's."""
    k = p.n[a] + 1
    (l0, r0, c0), (l1, r1, c1) = ([_cut(f, a, s, k) for f in par] for s in (0, 1))
    w = 1.0 - 2.0 * z / 3.0
    return r0 - 0.5 * z * (r0 - l0 - c0 * w), l1 + 0.5 * z * (r1 - l1 + c1 * w)


def _pressure(p, u):
    return p.isothermal ** 2 * u[0] if p.isothermal else (p.gamma - 1.0) * u[5]


def _step(p, u, mean):
    gam = 1.0 if p.isothermal else p.gamma
    hmin = min(p.h[: p.ndim])
    speed = torch.sqrt(sum((u[1 + a] / u[0]) ** 2 for a in range(p.ndim)))
    tau = p.cfl * hmin / (speed.max() + torch.sqrt(gam * _pressure(p, u) / u[0]).max())
    # Eulerian stage: acoustic Riemann problems on parabolas
    g = _ghosted(p, u)
    w = list(u)
    div_pv, div_v = torch.zeros_like(u[0]), torch.zeros_like(u[0])
    for a in range(p.ndim):
        n, h = p.n[a], p.h[a]
        rho = _line(p, g[0], a)
        s, v, pr = torch.sqrt(rho), _line(p, g[1 + a], a) / rho, _pressure(p, [_line(p, f, a) for f in g])
        A, B, C = ((_cut(f, a, 2, n + 1) + _cut(f, a, 3, n + 1)) for f in (rho * s, s, pr * s))
        lam, Z = torch.sqrt(gam * C / A), torch.sqrt(gam * A * C) / B
        z = lam * tau / h
        vm, vp = _strips(p, _parabolas(p, v, a), a, z)
        pm, pp = _strips(p, _parabolas(p, pr, a), a, z)
        V, P = 0.5 * (vm + vp) + (pm - pp) / (2.0 * Z), 0.5 * (pm + pp) + 0.5 * Z * (vm - vp)
        V0, V1, P0, P1 = _cut(V, a, 0, n), _cut(V, a, 1, n), _cut(P, a, 0, n), _cut(P, a, 1, n)
        w[1 + a] = u[1 + a] - tau * (P1 - P0) / h
        div_pv, div_v = div_pv + (P1 * V1 - P0 * V0) / h, div_v + (V1 - V0) / h
    w[4], w[5] = u[4] - tau * div_pv, u[5] - tau * (gam - 1.0) * u[5] * div_v
    grad = _force(p, u)
    if grad is not None:
        for a in range(p.ndim):
            w[1 + a], w[4] = w[1 + a] - tau * u[0] * grad[a], w[4] - tau * u[1 + a] * grad[a]
    # Lagrangian stage: upwind parabolic fluxes
    g = _ghosted(p, w)
    out = list(w)
    for a in range(p.ndim):
        n, h = p.n[a], p.h[a]
        vt = _cut(g[1 + a] / g[0], a, 2, n + 2)
        for o in range(p.ndim):
            if o != a:
                vt = 0.25 * (_cut(vt, o, 2, p.n[o]) + _cut(vt, o, 4, p.n[o])) + 0.5 * _cut(vt, o, 3, p.n[o])
        s = torch.sqrt(_cut(_line(p, g[0], a), a, 2, n + 2))
        s0, s1 = _cut(s, a, 0, n + 1), _cut(s, a, 1, n + 1)
        v = (_cut(vt, a, 0, n + 1) * s0 + _cut(vt, a, 1, n + 1) * s1) / (s0 + s1)
        z = v.abs() * tau / h
        for f in range(6):
            left, right = _strips(p, _parabolas(p, _line(p, g[f], a), a), a, z)
            F = v * torch.where(v >= 0, left, right)
            out[f] = out[f] - tau * (_cut(F, a, 1, n) - _cut(F, a, 0, n)) / h
    # total-energy correction
    rho, m2 = out[0], out[1] ** 2 + out[2] ** 2 + out[3] ** 2
    spare = out[4] - m2 / (2.0 * rho)
    thin = rho < (0.0 if p.isothermal else 1e-5) * mean
    kin = out[4] - out[5]
    scale = torch.where(kin > 0, torch.sqrt(2.0 * kin.clamp(min=0) * rho / m2.clamp(min=1e-300)), 0.0)
    e = torch.where(thin, torch.where((kin > 0) & (m2 > 0), out[5], out[4]), torch.where(spare > 0, spare, out[5]))
    return [rho, *(torch.where(thin, m * scale, m) for m in out[1:4]), out[4], e]


def _force(p, u):
    """Gradient of the fixed and the self-gravity potential at the cell centres."""
    grad = None
    if p.potential:
        X, Y, Z = _centres(p)
        kind, c = p.potential[0], p.potential[1:]
        if kind == "uniform":
            grad = list(c)
        elif kind == "log":
            k = c[0] ** 2 / (c[1] ** 2 + X * X + Y * Y + Z * Z / c[2] ** 2)
            grad = [k * X, k * Y, k * Z / c[2] ** 2]
        else:
            r = torch.sqrt(X * X + Y * Y + Z * Z).clamp(min=1e-300)
            q = torch.clamp(r, max=c[2]) / c[1]
            k = 4.0 * math.pi * c[0] * c[1] ** 3 * (q - torch.atan(q)) / r ** 3
            k = torch.where(r > 1e-200, k, 0.0)
            grad = [k * X, k * Y, k * Z]
    if p.self_gravity:
        phi = _potential(p, u[0])
        n = p.n
        for a in range(3):
            d = phi
            for o in range(3):
                d = _cut(d, o, 1, n[o]) if o != a else d
            d = (_cut(d, a, 2, n[a]) - _cut(d, a, 0, n[a])) / (2.0 * p.h[0])
            grad = grad or [0.0, 0.0, 0.0]
            grad[a] = grad[a] + d
    return grad


def _potential(p, rho):
    """27-point Poisson equation with multipole shell values, by sine transforms."""
    n, h, G, dev = p.n, p.h[0], p.self_gravity, rho.device
    X, Y, Z = _centres(p)
    m = rho * h ** 3
    M = m.sum()
    I = [((Y * Y + Z * Z) * m).sum(), ((X * X + Z * Z) * m).sum(), ((X * X + Y * Y) * m).sum()]
    ixy, ixz, iyz = (X * Y * m).sum(), (X * Z * m).sum(), (Y * Z * m).sum()
    x, y, z = (p.lo[a] + (torch.arange(-1, n[a] + 1, dtype=torch.float64, device=dev) + 0.5) * h for a in range(3))
    x, y, z = x[None, None, :], y[None, :, None], z[:, None, None]
    r2 = x * x + y * y + z * z
    i0 = (x * x * I[0] + y * y * I[1] + z * z * I[2] - 2.0 * (x * y * ixy + x * z * ixz + y * z * iyz)) / r2
    phi = -G * M / torch.sqrt(r2) - G * (I[0] + I[1] + I[2] - 3.0 * i0) / (2.0 * r2 * torch.sqrt(r2))
    phi[1:-1, 1:-1, 1:-1] = 0.0
    b = 4.0 * math.pi * G * h * h * rho
    for dz in range(3):
        for dy in range(3):
            for dx in range(3):
                k = (dz != 1) + (dy != 1) + (dx != 1)
                if k:
                    b = b - (4.0 / 9.0, 1.0 / 9.0, 1.0 / 36.0)[k - 1] * phi[dz: dz + n[2], dy: dy + n[1], dx: dx + n[0]]
    sines, factor = [], []
    for a in range(3):
        j = torch.arange(1, n[a] + 1, dtype=torch.float64, device=dev)
        sines.append(math.sqrt(2.0 / (n[a] + 1)) * torch.sin(math.pi * torch.remainder(j[:, None] * j, 2.0 * (n[a] + 1)) / (n[a] + 1)))
        factor.append(1.0 - 2.0 / 3.0 * torch.sin(math.pi * j / (2.0 * (n[a] + 1))) ** 2)

    def transform(f):
        f = (f.reshape(-1, n[0]) @ sines[0]).view(n[::-1])
        f = (f.transpose(1, 2).reshape(-1, n[1]) @ sines[1]).view(n[2], n[0], n[1]).transpose(1, 2)
        return (sines[2] @ f.reshape(n[2], -1)).view(n[::-1])

    lam = -6.0 * (1.0 - factor[0][None, None, :] * factor[1][None, :, None] * factor[2][:, None, None])
    phi[1:-1, 1:-1, 1:-1] = transform(transform(b) / lam)
    return phi


def _advance(p, steps):
    u = conserved(p)
    if p.ndim == 1:
        u = [f.cpu() for f in u]  # short lines: the launches would take longer than the work
    mean = u[0].mean()
    for _ in range(steps):
        u = _step(p, u, mean)
    return u


def exact(case, seed):
    if case["kind"] == "batch":
        out = []
        for c, sd in members(case, seed):
            p = problem(c, sd)
            u = _advance(p, case["steps"])
            out.append(torch.cat([f.flatten() for f in (*u[: 1 + p.ndim], *u[4:])]))
        return out
    p = problem(case, seed)
    if case["kind"] == "checkpoint":
        u = conserved(p)
        totals = np.array([float(f.sum()) for f in u])
        return {"totals": totals, "fields": [f.cpu().numpy() for f in u]}
    u = _advance(p, case["steps"])
    return {"rho": u[0], "mom": torch.stack(u[1: 1 + p.ndim]), "etot": u[4], "eint": u[5]}
