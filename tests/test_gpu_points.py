"""The FP64 point tile's two ways to finish a point -- the high-order state
taken as it is where a bound shows that no limiter can act, and the tile's
list of points whose first-order LLF state is formed -- at the edges of the
14 x 14 tiles, against the FP64 CPU oracle.

Tolerance: 1e-11 of each field's largest value, the single-stage bar of the
other parity tests, or, as where the round-off fallback acts, four times what
the oracle's own stage moves by when its input is perturbed by one ulp: a
shock that fills a 43 x 4 grid leaves limited pressures at round-off level
(1.6e-11 by the oracle itself).
"""
from dataclasses import replace

import numpy as np
import pytest

from paper_2506_04857_amd import inputs as I

pytestmark = pytest.mark.gpu

REL = 1e-11

# CFL 0.2: smooth points satisfy the bound, a shock's do not; CFL 0.9: the
# fastest points of every grid fail it
CASES = [(nx, ny, kind, bc, cfl)
         for nx, ny in ((14, 14), (15, 29), (28, 13), (43, 4))
         for kind, bc, cfl in (("smooth", I.PERIODIC, 0.2), ("smooth", I.OUTFLOW, 0.9), ("shock", I.OUTFLOW, 0.2),
                               ("shock", I.PERIODIC, 0.4))]


def problem(nx, ny, kind, bc, cfl):
    base = I.random_smooth(nx, ny, seed=nx, bc=bc) if kind == "smooth" else I.random_shock(nx, ny, seed=ny, bc=bc)
    return replace(I.stirred(base), cfl=cfl, kappa=0.0)


def worst(got, ref):
    return max(np.max(np.abs(g[k] - r[k])) / (np.max(np.abs(r[k])) or 1.0) for g, r in zip(got, ref) for k in range(8))


@pytest.mark.parametrize("nx,ny,kind,bc,cfl", CASES)
def test_point_tile_matches_oracle(oracle, nx, ny, kind, bc, cfl):
    import torch

    from oracle import oracle as O
    from paper_2506_04857_amd import af_mhd as af
    prob = problem(nx, ny, kind, bc, cfl)
    u = I.sample(prob)
    dt = oracle.dt(prob, u)
    c = O.Counters()
    ref = oracle.stage(prob, 0, u, u, dt, counters=c)
    ctx = af.Context(prob)
    ctx.dt_dev.fill_(dt)
    out = af.empty_state(prob)
    ctx.af_mhd_stage(0, af.to_device(u), af.to_device(u), out)
    st = ctx.af_mhd_stats(out)
    rng = np.random.default_rng(0)
    up = tuple(a * (1 + rng.choice([-1.0, 1.0], size=a.shape) * 2.0 ** -52) for a in u)
    bar = max(REL, 4 * worst(oracle.stage(prob, 0, up, up, dt), ref))
    assert worst(af.to_host(out), ref) <= bar
    assert st["n_point_limited"] == c.n_point_limited and st["n_llf_not_admissible"] == c.n_llf_not_admissible
    # in place on U^n, where listed points wait in the scratch state: the same bits
    un, un2, u2 = af.to_device(u), af.to_device(u), af.to_device(ref)
    ctx.af_mhd_stage(2, un, u2, out)
    ctx.af_mhd_stage(2, un2, u2, un2)
    torch.cuda.synchronize()
    ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(out, un2))
