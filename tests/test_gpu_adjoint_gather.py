"""The reverse of a stage on both sides of the point count from which the
points' lines are gathered (64000 points: 146 x 146 scatters, 147 x 147
periodic and 146 x 146 with outflow gather), on shock data with limited
points: the dot-product identity against the tangent oracle, bar 1e-10 as in
the adjoint's other tests."""
from dataclasses import replace

import numpy as np
import pytest

from paper_2506_04857_amd import inputs as I

pytestmark = pytest.mark.gpu

BAR = 1e-10


@pytest.mark.parametrize("n,bcx,bcy", [(146, I.PERIODIC, I.PERIODIC), (147, I.PERIODIC, I.PERIODIC),
                                       (146, I.OUTFLOW, I.OUTFLOW), (160, I.OUTFLOW, I.PERIODIC)])
def test_stage_dot_product(oracle, n, bcx, bcy):
    import torch

    from paper_2506_04857_amd import af_mhd as af
    prob = replace(I.stirred(I.random_shock(n, n, seed=4, bc=I.OUTFLOW)), bc_x=bcx, bc_y=bcy, x1=0.8)
    u0 = I.sample(prob)
    dt = oracle.dt(prob, u0)
    rng = np.random.default_rng(n)
    adj = af.Adjoint(prob)
    dt_dev = torch.full((1,), dt, dtype=torch.float64, device="cuda")
    uk, k = oracle.stage(prob, 0, u0, u0, dt), 1
    out, tape = af.empty_state(prob), adj.new_tape()
    adj.record(k, af.to_device(u0), af.to_device(uk), out, dt_dev, tape)
    lam = tuple(rng.standard_normal(a.shape) for a in u0)
    ln, lk = (tuple(torch.zeros_like(t) for t in out) for _ in range(2))
    adj.stage(k, af.to_device(uk), tape, dt_dev, af.to_device(lam), ln, lk)
    torch.cuda.synchronize()
    lkh = af.to_host(lk)
    v = tuple(rng.standard_normal(a.shape) for a in u0)
    _, d = oracle.tangent_stage(prob, k, u0, [tuple(np.zeros_like(a) for a in u0)], uk, [v], dt)
    gap = abs(sum(np.sum(a * b) for a, b in zip(lam, d[0])) - sum(np.sum(a * b) for a, b in zip(lkh, v)))
    print(f"[gather] {n} {bcx}{bcy} gap {gap:.2e}", flush=True)
    assert gap <= BAR * sum(np.sum(np.abs(a * b)) for a, b in zip(lam, d[0]))
    adj.close()
