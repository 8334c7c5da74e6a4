"""A recorded and reversed stage above the point count from which the points run
on an auxiliary stream beside the cells (160000: 240 x 240 with outflow holds
173761), on shock data with limited points and open boundaries: what the limited
points hand over, and the gather at the boundaries, cross from stream to stream.
The stage against the oracle's (1e-11 of each field's largest value, or four times
what the oracle's own stage moves by when its input is perturbed by one ulp, as in
the other parity tests), the reverse by the dot-product identity against the
tangent oracle, bar 1e-10 as in the adjoint's other tests."""
import numpy as np
import pytest

from paper_2506_04857_amd import inputs as I

pytestmark = pytest.mark.gpu

REL, BAR = 1e-11, 1e-10


def worst(got, ref):
    return max(np.max(np.abs(g[k] - r[k])) / (np.max(np.abs(r[k])) or 1.0) for g, r in zip(got, ref) for k in range(8))


@pytest.mark.parametrize("k", [0, 2])
def test_limited_stage_on_two_streams(oracle, k):
    import torch

    from oracle import oracle as O
    from paper_2506_04857_amd import af_mhd as af
    prob = I.stirred(I.random_shock(240, 240, seed=4, bc=I.OUTFLOW))
    u0 = I.sample(prob)
    dt = oracle.dt(prob, u0)
    uk = u0 if k == 0 else oracle.stage(prob, 0, u0, u0, dt)
    c = O.Counters()
    ref = oracle.stage(prob, k, u0, uk, dt, counters=c)
    assert c.n_point_limited > 0
    rng = np.random.default_rng(k)
    up = tuple(a * (1 + rng.choice([-1.0, 1.0], size=a.shape) * 2.0 ** -52) for a in uk)
    bar = max(REL, 4 * worst(oracle.stage(prob, k, up if k == 0 else u0, up, dt), ref))
    adj = af.Adjoint(prob)
    dt_dev = torch.full((1,), dt, dtype=torch.float64, device="cuda")
    dun, duk = af.to_device(u0), af.to_device(uk)
    out, tape = af.empty_state(prob), adj.new_tape()
    adj.record(k, dun, duk, out, dt_dev, tape)
    lam = tuple(rng.standard_normal(a.shape) for a in u0)
    ln, lk = (tuple(torch.zeros_like(t) for t in out) for _ in range(2))
    adj.stage(k, duk, tape, dt_dev, af.to_device(lam), ln if k else None, lk)
    torch.cuda.synchronize()
    adj.close()
    assert worst(af.to_host(out), ref) <= bar
    v = tuple(rng.standard_normal(a.shape) for a in u0)
    zero = tuple(np.zeros_like(a) for a in u0)
    _, d = oracle.tangent_stage(prob, k, u0, [v if k == 0 else zero], uk, [v], dt)
    gap = abs(sum(np.sum(a * b) for a, b in zip(lam, d[0])) - sum(np.sum(a * b) for a, b in zip(af.to_host(lk), v)))
    print(f"[two streams] k {k} limited {c.n_point_limited} gap {gap:.2e}", flush=True)
    assert gap <= BAR * sum(np.sum(np.abs(a * b)) for a, b in zip(lam, d[0]))
