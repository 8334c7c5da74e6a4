"""A stage in one launch (grids whose tiles all run at once) against the point
and cell launches, which a context with kernel timing keeps: the same bits, the
same counters, the same time steps.  The sizes: the smallest grid, one and two
cell tiles, and the largest tile counts that take one launch (256 at 291 x 100)."""
from dataclasses import replace

import pytest

from paper_2506_04857_amd import inputs as I

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bc", [I.PERIODIC, I.OUTFLOW])
@pytest.mark.parametrize("nx,ny", [(4, 4), (29, 13), (30, 14), (200, 137), (291, 100)])
def test_one_launch_is_bitwise_two_launches(nx, ny, bc):
    import torch

    from paper_2506_04857_amd import af_mhd as af
    prob = replace(I.stirred(I.random_shock(nx, ny, seed=nx, bc=bc)), kappa=1.0)
    u = I.sample(prob)
    got = []
    for flags in (0, af.AF_FLAG_KERNEL_TIMING):
        ctx = af.Context(prob, flags=flags | af.AF_FLAG_FUSED_DT)
        s, dts = af.to_device(u), []
        for _ in range(3):  # the last two take dt from the maxima that the step before left
            ctx.af_mhd_step(s)
            dts.append(float(ctx.dt_dev))
        out = af.empty_state(prob)
        ctx.af_mhd_stage(1, af.to_device(u), s, out)
        got.append((list(s) + list(out), dts, ctx.af_mhd_stats(s)))
        torch.cuda.synchronize()
        ctx.close()
    assert all(torch.equal(a, b) for a, b in zip(got[0][0], got[1][0]))
    assert got[0][1:] == got[1][1:]
