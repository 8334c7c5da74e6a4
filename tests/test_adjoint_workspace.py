"""The adjoint context asks for the memory that its launches use: the adjoints of
a stage's intermediates, and the lines' quantities only where the points' reverse
gathers them (more than 64000 points)."""
import ctypes

import pytest

from paper_2506_04857_amd import af_mhd as af
from paper_2506_04857_amd import inputs as I


def taken(*counts):
    return sum((8 * n + 255) // 256 * 256 for n in counts)


@pytest.mark.parametrize("nx,ny,bc,gather", [(4, 4, I.PERIODIC, False), (72, 50, I.OUTFLOW, False),
                                             (146, 146, I.PERIODIC, False), (147, 147, I.PERIODIC, True),
                                             (146, 146, I.OUTFLOW, True), (257, 100, I.OUTFLOW, True)])
def test_workspace(nx, ny, bc, gather):
    prob = I.random_shock(nx, ny, bc=bc)
    p = af.make_params(prob, 0)
    cells, ns, ne = nx * ny, (nx + 4) * (ny + 4), (nx + 2) * (ny + 2)
    xi, yi = (nx + 3) * (ny + 2), (nx + 2) * (ny + 3)
    want = taken(8 * cells, 4 * ns, 8 * xi, 8 * xi, xi, 8 * yi, 8 * yi, yi, 4 * ne, ne, 8 * ne, 8 * ne)
    if gather:
        for n in (prob.nxp * ny, nx * prob.nyp, prob.nxp * prob.nyp):
            want += taken(8 * n, 6 * n, (n + 1) // 2)
    assert af._lib.af_mhd_adj_workspace_bytes(ctypes.byref(p)) == want
