"""The work that programs built on this framework have it do, as cases that a
measuring program can prepare, run, and check against 64-bit arithmetic.

A case names a problem family, a grid and an entry point:
  step    Context.af_mhd_step: one SSP-RK3 step in place
  stages  Context.af_mhd_dt and three Context.af_mhd_stage, out of place
  loop    Solver.run: steps with the time advanced on the host
  batch   Batch.step: an ensemble of independent grids, one hipGraph per step
  evolve  evolve: some steps as a torch function, and the gradient of an
          objective of the end state with respect to the initial state
  divb    Context.af_mhd_divb: the two recorded divergences of a state

Inputs come from the seed: the set-ups of the repository (circularly polarised
Alfven wave, Orszag-Tang vortex, low-beta blast, random shock) with their
parameters varied and small smooth velocities and fields added, as in the middle
of a run (no region is at rest or free of discrete divergence to the last bit).

exact() is the scheme in plain torch, float64, one array operation at a time.
"""
from __future__ import annotations

import math
import random

import numpy as np
import torch

from paper_2506_04857_amd import af_mhd as af
from paper_2506_04857_amd import inputs

PERIODIC, OUTFLOW = inputs.PERIODIC, inputs.OUTFLOW
ENSEMBLE_SIZES = inputs.BATCH_SIZES
EPS = 1e-13  # lower bounds of the positivity limiters

# bytes of one stage per cell: U^(k) and (two of three stages) U^n read, the
# output written, four sets of eight doubles each; operations of one stage per
# cell, each flux, wave speed and limiter test counted once
STAGE_BYTES = (512 + 768 + 768) / 3.0
STAGE_FLOPS = 4000.0


def listed():
    return [
        # the smallest grid of the repository's configurations: a step is launches and their latency
        {"name": "alfven_32_step", "entry": "step", "problem": "alfven", "nx": 32, "ny": 32},
        # a time loop on the host that reads every dt back, as the accuracy and convergence tests are run
        {"name": "alfven_64_loop", "entry": "loop", "problem": "alfven", "nx": 64, "ny": 64, "steps": 10},
        # a ragged grid with open boundaries, stepped out of place by the stage calls (a caller's own integrator)
        {"name": "shock_200x137_stages", "entry": "stages", "problem": "shock", "nx": 200, "ny": 137},
        # the ordinary production size, periodic
        {"name": "orszag_tang_512_step", "entry": "step", "problem": "orszag_tang", "nx": 512, "ny": 512,
         "fused_dt": True},
        # the benchmark workload
        {"name": "blast_1024_step", "entry": "step", "problem": "blast", "nx": 1024, "ny": 1024, "fused_dt": True},
        # the same with the FP32-bulk option
        {"name": "blast_1024_fp32_step", "entry": "step", "problem": "blast", "nx": 1024, "ny": 1024,
         "fused_dt": True, "fp32": True},
        # the largest single grid
        {"name": "blast_2048_step", "entry": "step", "problem": "blast", "nx": 2048, "ny": 2048, "fused_dt": True},
        # a small ensemble: too few tiles to fill the device by itself
        {"name": "ensemble_8_step", "entry": "batch", "problem": "orszag_tang", "count": 8, "sizes_seed": 8},
        # the ensemble of the benchmark
        {"name": "ensemble_256_step", "entry": "batch", "problem": "orszag_tang", "count": 256, "sizes_seed": 256},
        # the gradient workload's grid, a few steps of it: recording forward and reverse sweep
        {"name": "alfven_256_evolve", "entry": "evolve", "problem": "alfven", "nx": 256, "ny": 256, "steps": 4},
        # a small, ragged gradient with open boundaries and active limiters
        {"name": "shock_72x50_evolve", "entry": "evolve", "problem": "shock", "nx": 72, "ny": 50, "steps": 3},
        # the divergence record of a run (the set-up's 400 x 400 grid)
        {"name": "orszag_tang_400_divb", "entry": "divb", "problem": "orszag_tang", "nx": 400, "ny": 400},
    ]


def draw(rng):
    def size(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    entry = rng.choice(["step", "step", "step", "stages", "loop", "batch", "batch", "evolve", "divb"])
    if entry == "batch":
        return {"entry": entry, "problem": "orszag_tang", "count": size(2, 128), "sizes_seed": rng.randrange(1 << 20),
                "fp32": rng.random() < 0.2}
    problem = rng.choice(["alfven", "orszag_tang", "blast", "shock"])
    if entry == "divb":
        return {"entry": entry, "problem": problem, "nx": size(32, 1024), "ny": size(32, 1024)}
    if entry == "evolve":
        return {"entry": entry, "problem": rng.choice(["alfven", "orszag_tang", "shock"]), "nx": size(32, 200),
                "ny": size(32, 200), "steps": rng.randint(1, 4)}
    if entry == "loop":
        return {"entry": entry, "problem": problem, "nx": size(32, 128), "ny": size(32, 128),
                "steps": rng.randint(2, 10)}
    case = {"entry": entry, "problem": problem, "nx": size(32, 1024), "ny": size(32, 1024)}
    if entry == "step":
        case["fused_dt"] = rng.random() < 0.6
        case["fp32"] = rng.random() < 0.2
    return case


# ------------------------------------------------------------------ inputs
def _waves(rng, lx, ly, n=3):
    """A smooth seeded field of unit size on an lx x ly periodic box."""
    q = [(rng.randint(1, 3), rng.randint(1, 3), rng.uniform(0, 2 * math.pi), rng.uniform(0.5, 1.0) / n)
         for _ in range(n)]

    def f(x, y):
        return sum(a * torch.sin(2 * math.pi * (m * x / lx + k * y / ly) + ph) for m, k, ph, a in q)

    return f


def _problem(case, seed, nx, ny):
    """(inputs.Problem, prim(x, y) -> eight primitive fields)."""
    rng = random.Random(seed * 7919 + nx * 131 + ny)
    kind = case["problem"]
    if kind == "alfven":
        p = inputs.alfven(nx).with_size(nx, ny)
        lx, ly = p.x1 - p.x0, p.y1 - p.y0
        d = [_waves(rng, lx, ly) for _ in range(4)]
        ph0 = rng.uniform(0, 2 * math.pi)
        r2 = math.sqrt(0.5)

        def prim(x, y):
            ph = 2 * math.pi * r2 * (x + y) + ph0
            s, c = 0.1 * torch.sin(ph), 0.1 * torch.cos(ph)
            one = torch.ones_like(x)
            return [one + 1e-3 * d[0](x, y), -r2 * s + 1e-3 * d[1](x, y), r2 * s + 1e-3 * d[2](x, y), c,
                    r2 * (1 - s) + 1e-3 * d[3](x, y), r2 * (1 + s), c, 0.1 * one]
    elif kind == "orszag_tang":
        p = inputs.orszag_tang(nx).with_size(nx, ny)
        lx = ly = 2 * math.pi
        d = [_waves(rng, lx, ly) for _ in range(5)]
        z = [1 + 0.05 * rng.gauss(0, 1) for _ in range(8)]
        g = 5.0 / 3.0

        def prim(x, y):
            one, zero = torch.ones_like(x), torch.zeros_like(x)
            return [z[0] * g * g * (one + 0.02 * d[0](x, y)), -z[1] * torch.sin(y) + 0.05 * d[1](x, y),
                    z[2] * torch.sin(x) + 0.05 * d[2](x, y), zero, -z[4] * torch.sin(y) + 0.005 * d[3](x, y),
                    z[5] * torch.sin(2 * x) + 0.005 * d[4](x, y), zero, z[7] * g * one]
    else:
        p = (inputs.blast_lowbeta(nx) if kind == "blast" else inputs.random_shock(nx, ny, bc=OUTFLOW)).with_size(nx, ny)
        lx, ly = p.x1 - p.x0, p.y1 - p.y0
        d = [_waves(rng, lx, ly) for _ in range(5)]
        cx, cy = p.x0 + lx * rng.uniform(0.4, 0.6), p.y0 + ly * rng.uniform(0.4, 0.6)
        r0 = 0.1 * rng.uniform(0.9, 1.1) * (1.0 if kind == "blast" else 2.0)
        pin = (1000.0 if kind == "blast" else 100.0) * rng.uniform(0.9, 1.1)
        if kind == "blast":
            rho, b, pout = (1.0, 1.0), (100.0 / math.sqrt(4 * math.pi), 0.0, 0.0), 0.1
        else:
            rho, b, pout = (1.0, 0.125), [rng.uniform(1, 5) * rng.choice((-1, 1)) for _ in range(3)], 0.1

        bd = 0.002 * max(abs(t) for t in b)

        def prim(x, y):
            one = torch.ones_like(x)
            ins = (x - cx) ** 2 + ((y - cy) * lx / ly) ** 2 < r0 * r0
            return [torch.where(ins, rho[0] * one, rho[1] * one) * (one + 0.02 * d[0](x, y)), 0.2 * d[1](x, y),
                    0.2 * d[2](x, y), 0 * one, b[0] * one + bd * d[3](x, y), b[1] * one + bd * d[4](x, y), b[2] * one,
                    torch.where(ins, pin * one, pout * one)]
    return p, prim


def _cons(w, gamma):
    rho, v1, v2, v3, b1, b2, b3, p = w
    e = p / (gamma - 1) + 0.5 * rho * (v1 * v1 + v2 * v2 + v3 * v3) + 0.5 * (b1 * b1 + b2 * b2 + b3 * b3)
    return torch.stack([rho, rho * v1, rho * v2, rho * v3, b1, b2, b3, e])


def _sample(p, prim, device):
    """Point values at their places, cell averages by a 3 x 3 Gauss rule."""
    def axis(n, a, d, off):
        return a + (torch.arange(n, dtype=torch.float64, device=device) + off) * d

    def at(xs, ys):
        y, x = torch.meshgrid(ys, xs, indexing="ij")
        return _cons(prim(x, y), p.gamma)

    g = math.sqrt(0.6) / 2
    cell = 0.0
    for a, wa in ((-g, 5.0 / 18), (0.0, 8.0 / 18), (g, 5.0 / 18)):
        for b, wb in ((-g, 5.0 / 18), (0.0, 8.0 / 18), (g, 5.0 / 18)):
            cell = cell + wa * wb * at(axis(p.nx, p.x0, p.dx, 0.5 + a), axis(p.ny, p.y0, p.dy, 0.5 + b))
    xc, yc = axis(p.nx, p.x0, p.dx, 0.5), axis(p.ny, p.y0, p.dy, 0.5)
    xn, yn = axis(p.nxp, p.x0, p.dx, 0.0), axis(p.nyp, p.y0, p.dy, 0.0)
    return tuple(t.contiguous() for t in (cell, at(xn, yc), at(xc, yn), at(xn, yn)))


def _members(case):
    """Grid sizes of the case's grids: one, or an ensemble's."""
    if case["entry"] != "batch":
        return [(case["nx"], case["ny"])]
    rng = random.Random(case["sizes_seed"])
    return [(rng.choice(ENSEMBLE_SIZES), rng.choice(ENSEMBLE_SIZES)) for _ in range(case["count"])]


def _inputs(case, seed, device):
    """[(problem, state)] of the case's grids."""
    got = []
    for m, (nx, ny) in enumerate(_members(case)):
        p, prim = _problem(case, seed + 1009 * m, nx, ny)
        got.append((p, _sample(p, prim, device)))
    return got


def _flags(case):
    return (af.AF_FLAG_FP32_BULK if case.get("fp32") else 0) | (af.AF_FLAG_FUSED_DT if case.get("fused_dt") else 0)


def prepare(case, seed):
    got = _inputs(case, seed, "cuda")
    s = {"entry": case["entry"], "steps": case.get("steps", 1)}
    if case["entry"] == "batch":
        # the ensemble's states in one allocation, as a program that writes it out whole keeps them
        arena = torch.empty(sum(t.numel() for _, u in got for t in u), dtype=torch.float64, device="cuda")
        states, at = [], 0
        for _, u in got:
            views = []
            for t in u:
                view = arena[at:at + t.numel()].view(t.shape)
                view.copy_(t)
                views.append(view)
                at += t.numel()
            states.append(tuple(views))
        s["arena"] = arena
        s["batch"] = af.Batch([p for p, _ in got], states, flags=_flags(case))
        return s
    p, u = got[0]
    s["problem"], s["u"] = p, u
    if case["entry"] == "evolve":
        s["u"] = tuple(t.requires_grad_() for t in u)
    elif case["entry"] == "loop":
        s["solver"] = af.Solver(p)
    else:
        s["ctx"] = af.Context(p, flags=_flags(case))
        if case["entry"] == "stages":
            s["buffers"] = [af.empty_state(p) for _ in range(3)]
    return s


def run(s):
    entry = s["entry"]
    if entry == "step":
        return list(s["ctx"].af_mhd_step(s["u"]))
    if entry == "stages":
        ctx, u = s["ctx"], s["u"]
        u1, u2, out = s["buffers"]
        dt = ctx.af_mhd_dt(u)
        ctx.af_mhd_stage(0, u, u, u1)
        ctx.af_mhd_stage(1, u, u1, u2)
        ctx.af_mhd_stage(2, u, u2, out)
        return list(out) + [dt]
    if entry == "loop":
        t, n = s["solver"].run(s["u"], 1e9, max_steps=s["steps"])
        return list(s["u"]) + [t, n]
    if entry == "batch":
        s["batch"].step()
        return [s["arena"]]
    if entry == "evolve":
        out = af.evolve(s["problem"], s["u"], s["steps"])
        objective = 0.5 * torch.sum((out[0][0] - 1.0) ** 2)
        return [t.detach() for t in out] + list(torch.autograd.grad(objective, s["u"]))
    return s["ctx"].af_mhd_divb(s["u"])


def work(case):
    cells = float(sum(nx * ny for nx, ny in _members(case)))
    if case["entry"] == "divb":
        return {"bytes": 256 * cells, "flops": 250 * cells}
    stages = 3 * case.get("steps", 1)
    # the reverse sweep reads the stage inputs and the adjoints and writes adjoints: three times the forward's
    reverse = 4 if case["entry"] == "evolve" else 1
    return {"bytes": reverse * stages * STAGE_BYTES * cells, "flops": reverse * stages * STAGE_FLOPS * cells}


# --------------------------------------------------- the scheme in 64 bits
PAD = 3


def _index(n, count, outflow, node, device):
    """Source indices of the entries -PAD .. count-1+PAD of one direction."""
    k = np.arange(-PAD, count + PAD)
    if not outflow:
        k %= n
    elif node:
        k = np.where(k < 0, -k, np.where(k > n, 2 * n - k, k))
    else:
        k = np.where(k < 0, -1 - k, np.where(k >= n, 2 * n - 1 - k, k))
    return torch.as_tensor(k, device=device)


def _extend(p, u):
    """The four sets with PAD cells around, as the boundaries continue them:
    cells -PAD .. n+PAD-1 and nodes -PAD .. n+PAD of each direction."""
    ox, oy, dev = p.bc_x == OUTFLOW, p.bc_y == OUTFLOW, u[0].device
    cx, cy = _index(p.nx, p.nx, ox, False, dev), _index(p.ny, p.ny, oy, False, dev)
    kx, ky = _index(p.nx, p.nx + 1, ox, True, dev), _index(p.ny, p.ny + 1, oy, True, dev)
    return (u[0][:, cy][:, :, cx], u[1][:, cy][:, :, kx], u[2][:, ky][:, :, cx], u[3][:, ky][:, :, kx])


def _sq(u, a):
    return u[a] * u[a] + u[a + 1] * u[a + 1] + u[a + 2] * u[a + 2]


def _pressure(u, gamma):
    return (gamma - 1) * (u[7] - _sq(u, 1) / (2 * u[0]) - _sq(u, 4) / 2)


def _root(x):
    """sqrt with derivative 0 at 0."""
    ok = x > 0
    return torch.where(ok, torch.sqrt(torch.where(ok, x, torch.ones_like(x))), torch.zeros_like(x))


def _speeds(u, gamma, d):
    """Normal velocity and fast speed."""
    c2, b2 = gamma * _pressure(u, gamma) / u[0], _sq(u, 4) / u[0]
    s = c2 + b2
    disc = torch.clamp(s * s - 4 * c2 * u[4 + d] ** 2 / u[0], min=0.0)
    return u[1 + d] / u[0], _root(0.5 * (s + _root(disc)))


def _flux(u, gamma, d):
    v, b = u[1:4] / u[0], u[4:7]
    pt = _pressure(u, gamma) + _sq(u, 4) / 2
    vb = v[0] * b[0] + v[1] * b[1] + v[2] * b[2]
    f = [u[0] * v[d]] + [u[0] * v[d] * v[k] - b[d] * b[k] + (pt if k == d else 0.0) for k in range(3)]
    f += [v[d] * b[k] - b[d] * v[k] if k != d else torch.zeros_like(pt) for k in range(3)]
    return torch.stack(f + [(u[7] + pt) * v[d] - b[d] * vb])


def _psi(u):
    v = u[1:4] / u[0]
    return torch.cat([torch.zeros_like(u[:1]), u[4:7], v, (v * u[4:7]).sum(0, keepdim=True)])


def _llf(a, b, gamma, d):
    """LLF flux between the states a and b, the Lemma's viscosity."""
    va, ca = _speeds(a, gamma, d)
    vb, cb = _speeds(b, gamma, d)
    ra, rb = torch.sqrt(a[0]), torch.sqrt(b[0])
    jump = _root(_sq(a - b, 4)) / (ra + rb)
    roe = (ra * va + rb * vb).abs() / (ra + rb)
    al = torch.maximum(torch.maximum(va.abs(), vb.abs()), roe) + torch.maximum(ca, cb) + jump
    al = torch.maximum(al, torch.maximum(va.abs() + ca, vb.abs() + cb))
    return 0.5 * (_flux(a, gamma, d) + _flux(b, gamma, d) - al * (b - a))


def _fvs(w, gamma, d, h):
    """D+F+ + D-F- over the five states of a line, and its normal-field part."""
    al = None
    for u in w:
        v, c = _speeds(u, gamma, d)
        al = v.abs() + c if al is None else torch.maximum(al, v.abs() + c)
    f = [_flux(u, gamma, d) for u in w]
    r = (f[0] - 4 * f[1] + 4 * f[3] - f[4] + al * (w[0] - 4 * w[1] + 6 * w[2] - 4 * w[3] + w[4])) / (2 * h)
    b = 4 + d
    return r, (w[0][b] - 4 * w[1][b] + 4 * w[3][b] - w[4][b]) / (2 * h)


def _guard(act, num, den):
    """num / den where act holds, else 1."""
    return torch.where(act, num / torch.where(act, den, torch.ones_like(den)), torch.ones_like(num))


def _scale(uh, ul, gamma, whole):
    """Scaling limiter of uh towards ul: density step (the whole state for the
    centre value, the density alone for a point), then pressure step."""
    pl = _pressure(ul, gamma)
    er, ep = torch.clamp(ul[0], max=EPS), torch.clamp(pl, max=EPS)
    t1 = _guard(uh[0] < er, ul[0] - er, ul[0] - uh[0])
    us = t1 * uh + (1 - t1) * ul if whole else torch.cat([(t1 * uh[0] + (1 - t1) * ul[0])[None], uh[1:]])
    ps = _pressure(us, gamma)
    t2 = _guard(ps < ep, pl - ep, pl - ps)
    return t2 * us + (1 - t2) * ul


def _centres(e, gamma):
    a, x, y, v = e
    faces = (x[:, :, :-1] + x[:, :, 1:]) + (y[:, :-1] + y[:, 1:])
    corners = (v[:, :-1, :-1] + v[:, :-1, 1:]) + (v[:, 1:, :-1] + v[:, 1:, 1:])
    return _scale((36 * a - 4 * faces - corners) / 16, a, gamma, True)


def _points(p, e, c, dt):
    """Limited forward-Euler update of the three point sets."""
    a, x, y, v = e
    gamma = p.gamma
    ends = {"x": (p.nxp, p.ny), "y": (p.nx, p.nyp), "v": (p.nxp, p.nyp)}

    def pick(t, which, i, j):
        w, h = ends[which]
        return t[:, PAD + j:PAD + j + h, PAD + i:PAD + i + w]

    out = {}
    for which, own in (("x", x), ("y", y), ("v", v)):
        def at(t, i, j, which=which):
            return pick(t, which, i, j)

        u = at(own, 0, 0)
        mid = {"x": c, "y": v, "v": y}[which]  # halfway along x
        off = 1 if which == "y" else 0
        if which == "y":  # central in x between the vertices
            wl, wr = at(v, 0, 0), at(v, 1, 0)
            rx, bx = (_flux(wr, gamma, 0) - _flux(wl, gamma, 0)) / p.dx, (wr[4] - wl[4]) / p.dx
        else:
            wl, wr = at(own, -1, 0), at(own, 1, 0)
            rx, bx = _fvs([wl, at(mid, -1, 0), u, at(mid, off, 0), wr], gamma, 0, p.dx)
        if which == "x":  # central in y between the vertices
            wd, wu = at(v, 0, 0), at(v, 0, 1)
            ry, by = (_flux(wu, gamma, 1) - _flux(wd, gamma, 1)) / p.dy, (wu[5] - wd[5]) / p.dy
        else:
            mid = c if which == "y" else x
            wd, wu = at(own, 0, -1), at(own, 0, 1)
            ry, by = _fvs([wd, at(mid, 0, -1), u, at(mid, 0, 0), wu], gamma, 1, p.dy)
        psi = _psi(u)
        uh = u + dt * (-rx - ry - (bx + by) * psi)
        div = (wr[4] - wl[4]) / (2 * p.dx) + (wu[5] - wd[5]) / (2 * p.dy)
        ul = (u - dt / p.dx * (_llf(u, wr, gamma, 0) - _llf(wl, u, gamma, 0))
              - dt / p.dy * (_llf(u, wu, gamma, 1) - _llf(wd, u, gamma, 1)) - dt * div * psi)
        out[which] = _scale(uh, ul, gamma, False)
    return out["x"], out["y"], out["v"]


def _d3(at, u0, u1, u2):
    return (-3 * u0 + 4 * u1 - u2) if at == 0 else (u2 - u0) if at == 1 else (u0 - 4 * u1 + 3 * u2)


def _source(p, e, c):
    """Nine-point source of every extended cell."""
    _, x, y, v = e
    s9 = [[v[:, :-1, :-1], x[:, :, :-1], v[:, 1:, :-1]], [y[:, :-1], c, y[:, 1:]],
          [v[:, :-1, 1:], x[:, :, 1:], v[:, 1:, 1:]]]  # [along x][along y]
    w, s = (1 / 6, 2 / 3, 1 / 6), 0.0
    for i in range(3):
        for j in range(3):
            div = (_d3(i, *(s9[k][j][4] for k in range(3))) / p.dx + _d3(j, *(s9[i][k][5] for k in range(3))) / p.dy)
            s = s + w[i] * w[j] * div * _psi(s9[i][j])
    return s


def _sensor(p, a):
    """phi1x, phi1y, phi2, phi3 of the extended cells but the outermost ring."""
    pt, v, b = _pressure(a, p.gamma) + _sq(a, 4) / 2, a[1:3] / a[0], a[4:6]

    def sh(t, i, j):
        return t[..., 1 + j:t.shape[-2] - 1 + j, 1 + i:t.shape[-1] - 1 + i]

    def jameson(lo, hi):
        return (hi - 2 * sh(pt, 0, 0) + lo).abs() / (hi + 2 * sh(pt, 0, 0) + lo).abs()

    dv = (sh(v, 1, 0) - sh(v, -1, 0)) / (2 * p.dx), (sh(v, 0, 1) - sh(v, 0, -1)) / (2 * p.dy)
    div, curl = dv[0][0] + dv[1][1], dv[0][1] - dv[1][0]
    phi2 = torch.clamp(-div / torch.sqrt(div * div + curl * curl + 1e-40), min=0.0)
    db = sh(b, 1, 0)[0] - sh(b, -1, 0)[0] + sh(b, 0, 1)[1] - sh(b, 0, -1)[1]
    phi3 = db.abs() / (sh(b, 0, 0)[0] + sh(b, 0, 0)[1]).abs().add(1e-40)
    return jameson(sh(pt, -1, 0), sh(pt, 1, 0)), jameson(sh(pt, 0, -1), sh(pt, 0, 1)), phi2, phi3


def _cubic(a1, d, r, gamma, ep):
    w = a1 + r * d
    en = w[7] - _sq(w, 4) / 2 - ep / (gamma - 1)
    q = w[0] * en - _sq(w, 1) / 2
    dq = d[0] * en + w[0] * (d[7] - (w[4:7] * d[4:7]).sum(0)) - (w[1:4] * d[1:4]).sum(0)
    return q, dq


def _vertex_root(a1, d, gamma, ep):
    """Root of the pressure condition along a1 + r d, from r = 1 inside a sign
    bracket; its derivative by one more Newton step."""
    with torch.no_grad():
        lo, hi, r = torch.zeros_like(ep), torch.ones_like(ep), torch.ones_like(ep)
        done = torch.zeros_like(ep, dtype=torch.bool)
        for _ in range(50):
            q, dq = _cubic(a1, d, r, gamma, ep)
            lo, hi = torch.where(q >= 0, r, lo), torch.where(q >= 0, hi, r)
            rn = r - q / dq
            rn = torch.where((rn >= lo) & (rn <= hi), rn, 0.5 * (lo + hi))
            step = (rn - r).abs()
            r = torch.where(done, r, rn)
            done = done | (step <= 1e-13)
            if bool(done.all()):
                break
        dq = _cubic(a1, d, r, gamma, ep)[1]
    if not (a1.requires_grad or d.requires_grad):
        return r
    q = _cubic(a1, d, r, gamma, ep)[0]
    return r - (q - q.detach()) / dq


def _box(a1, h, gamma, er, ep):
    """Lambda of the four interfaces: density box, pressure at its vertices."""
    neg = sum(torch.clamp(t[0], max=0.0) for t in h)
    lr = [torch.clamp(_guard(t[0] < 0, a1[0] - er, 1e-12 - neg), max=1.0) for t in h]
    rmin = [torch.ones_like(neg) for _ in h]
    for k in range(1, 16):
        d = sum(lr[i] * h[i] for i in range(4) if k >> i & 1)
        bad = _pressure(a1 + d, gamma) < ep
        if bool(bad.any()):
            at = bad.nonzero(as_tuple=True)
            r = torch.ones_like(neg).index_put(at, _vertex_root(a1[:, at[0], at[1]], d[:, at[0], at[1]], gamma, ep[at]))
            for i in range(4):
                if k >> i & 1:
                    rmin[i] = torch.minimum(rmin[i], r)
    return [lr[i] * rmin[i] for i in range(4)]


def _cells(p, e, c, dt):
    """Limited forward-Euler update of the cell averages."""
    a, x, y, v = e
    gamma, nx, ny = p.gamma, p.nx, p.ny
    phi = _sensor(p, a)  # cells [-2, n+2)
    lx, ly = dt / p.dx, dt / p.dy

    def theta(q, lo, hi):
        m = [torch.maximum(t[lo], t[hi]) for t in (phi[q], phi[2], phi[3])]
        return torch.exp(-p.kappa * (m[0] * m[1] + m[2]))

    # interfaces of the cells [-1, n+1): x-interfaces k in [-1, n+2), rows [-1, n+1)
    r1 = slice(1, -1)
    tx = theta(0, (r1, slice(0, -1)), (r1, slice(1, None)))
    ty = theta(1, (slice(0, -1), r1), (slice(1, None), r1))
    cy, cx = slice(PAD - 1, PAD + ny + 1), slice(PAD - 1, PAD + nx + 1)
    fv = _flux(v, gamma, 0)[:, PAD - 1:PAD + ny + 2, PAD - 1:PAD + nx + 2]
    sx = (fv[:, :-1] + 4 * _flux(x[:, cy, PAD - 1:PAD + nx + 2], gamma, 0) + fv[:, 1:]) / 6
    fl_x = _llf(a[:, cy, PAD - 2:PAD + nx + 1], a[:, cy, PAD - 1:PAD + nx + 2], gamma, 0)
    fv = _flux(v, gamma, 1)[:, PAD - 1:PAD + ny + 2, PAD - 1:PAD + nx + 2]
    sy = (fv[:, :, :-1] + 4 * _flux(y[:, PAD - 1:PAD + ny + 2, cx], gamma, 1) + fv[:, :, 1:]) / 6
    fl_y = _llf(a[:, PAD - 2:PAD + ny + 1, cx], a[:, PAD - 1:PAD + ny + 2, cx], gamma, 1)
    dfx, dfy = tx * (sx - fl_x), ty * (sy - fl_y)
    aa = a[:, cy, cx]
    s_hi = _source(p, e, c)[:, cy, cx]
    div = ((a[4, cy, PAD:PAD + nx + 2] - a[4, cy, PAD - 2:PAD + nx]) / (2 * p.dx)
           + (a[5, PAD:PAD + ny + 2, cx] - a[5, PAD - 2:PAD + ny, cx]) / (2 * p.dy))
    s_lo = div * _psi(aa)
    tmin = torch.minimum(torch.minimum(tx[:, :-1], tx[:, 1:]), torch.minimum(ty[:-1], ty[1:]))
    s_s = tmin * s_hi + (1 - tmin) * s_lo
    g = aa - lx * (fl_x[:, :, 1:] - fl_x[:, :, :-1]) - ly * (fl_y[:, 1:] - fl_y[:, :-1])
    a_llf, a_src = g - dt * s_lo, g - dt * s_s
    pl, ps = _pressure(a_llf, gamma), _pressure(a_src, gamma)
    er, ep = torch.clamp(a_llf[0], max=EPS), torch.clamp(pl, max=EPS)
    ths = _guard(ps < ep, pl - ep, pl - ps)
    a1 = ths * a_src + (1 - ths) * a_llf
    h = [lx * dfx[:, :, :-1], -lx * dfx[:, :, 1:], ly * dfy[:, :-1], -ly * dfy[:, 1:]]
    lam = _box(a1, h, gamma, er, ep)
    thx = torch.minimum(lam[1][1:-1, :-1], lam[0][1:-1, 1:])  # x-interfaces [0, nx], rows of the grid
    thy = torch.minimum(lam[3][:-1, 1:-1], lam[2][1:, 1:-1])
    fx = fl_x[:, 1:-1, 1:-1] + thx * dfx[:, 1:-1, 1:-1]
    fy = fl_y[:, 1:-1, 1:-1] + thy * dfy[:, 1:-1, 1:-1]
    s = (ths * s_s + (1 - ths) * s_lo)[:, 1:-1, 1:-1]
    old = a[:, PAD:PAD + ny, PAD:PAD + nx]
    return old - lx * (fx[:, :, 1:] - fx[:, :, :-1]) - ly * (fy[:, 1:] - fy[:, :-1]) - dt * s


def _forward_euler(p, u, dt):
    e = _extend(p, u)
    c = _centres(e, p.gamma)
    return (_cells(p, e, c, dt),) + _points(p, e, c, dt)


def _time_step(p, u):
    mx = 0.0
    for t in u:
        (v1, c1), (v2, c2) = _speeds(t.detach(), p.gamma, 0), _speeds(t.detach(), p.gamma, 1)
        mx = max(mx, float(((v1.abs() + c1) / p.dx + (v2.abs() + c2) / p.dy).max()))
    return p.cfl / mx


def _step(p, u):
    dt = _time_step(p, u)
    u1 = _forward_euler(p, u, dt)
    u2 = tuple(0.75 * a + 0.25 * b for a, b in zip(u, _forward_euler(p, u1, dt)))
    return tuple(a / 3.0 + 2.0 / 3.0 * b for a, b in zip(u, _forward_euler(p, u2, dt))), dt


def _divb(p, u):
    e = _extend(p, u)
    c = _centres(e, p.gamma)
    _, x, y, v = e
    s9 = [[v[:, :-1, :-1], x[:, :, :-1], v[:, 1:, :-1]], [y[:, :-1], c, y[:, 1:]],
          [v[:, :-1, 1:], x[:, :, 1:], v[:, 1:, 1:]]]
    w, one, inner = (1 / 6, 2 / 3, 1 / 6), 0.0, (slice(PAD, PAD + p.ny), slice(PAD, PAD + p.nx))
    for i in range(3):
        for j in range(3):
            div = (_d3(i, *(s9[k][j][4] for k in range(3))) / p.dx + _d3(j, *(s9[i][k][5] for k in range(3))) / p.dy)
            one = one + w[i] * w[j] * div.abs()

    def edge(b, pts):
        return pts[0][b] + 4 * pts[1][b] + pts[2][b]

    top, bottom = [s9[k][2] for k in range(3)], [s9[k][0] for k in range(3)]
    two = edge(4, s9[2]) - edge(4, s9[0]) + edge(5, top) - edge(5, bottom)
    return torch.stack([one[inner].sum(), two[inner].abs().sum() / 6]) * (p.dx * p.dy)


def exact(case, seed, device="cuda"):
    got = _inputs(case, seed, device)
    if case["entry"] == "batch":
        with torch.no_grad():
            return [torch.cat([t.reshape(-1) for p, u in got for t in _step(p, u)[0]])]
    p, u = got[0]
    if case["entry"] == "evolve":
        u = tuple(t.requires_grad_() for t in u)
        out = u
        for _ in range(case["steps"]):
            out = _step(p, out)[0]
        objective = 0.5 * torch.sum((out[0][0] - 1.0) ** 2)
        return [t.detach() for t in out] + list(torch.autograd.grad(objective, u))
    with torch.no_grad():
        if case["entry"] == "divb":
            return _divb(p, u)
        t = 0.0
        for _ in range(case.get("steps", 1)):
            u, dt = _step(p, u)
            t += dt
    if case["entry"] == "stages":
        return list(u) + [torch.full((1,), t, dtype=torch.float64)]
    return list(u) + ([t, case["steps"]] if case["entry"] == "loop" else [])
