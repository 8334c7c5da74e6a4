"""The points' reverse as the kernels run it (line quantities, then one gather
a DoF) against the scatter form, on the host: every mix of boundaries, the
smallest grids and odd ones, limited points, and an adjoint with zeros in it.
The two sum the same products in another order; the bar is that of the
adjoint's dot-product tests, 1e-11 of each component's largest entry."""
import ctypes
import os
import subprocess
import sys
from dataclasses import replace

import numpy as np
import pytest

from paper_2506_04857_amd import inputs as I

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from hostcheck import hostcheck as hc  # noqa: E402

BAR = 1e-11


@pytest.fixture(scope="module")
def points(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("gather") / "libgather.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", hc.CSRC,
                           os.path.join(hc.HERE, "adjoint_gather_check.cpp"), "-o", out])
    fn = ctypes.CDLL(out).hc_points
    fn.argtypes = [ctypes.POINTER(hc._P), ctypes.c_int, hc._DD, ctypes.c_void_p, ctypes.c_double, hc._DD, hc._DD,
                   hc._DD, hc._D, ctypes.c_void_p, ctypes.c_int]
    fn.restype = None

    def run(prob, k, uk, tape, dt, lam, gather):
        p = hc._params(prob)
        ln, lk = (tuple(np.zeros_like(a) for a in uk) for _ in range(2))
        lc = np.zeros((8, prob.ny, prob.nx))
        buf = np.zeros(hc.lib().hc_adjbuf_bytes(ctypes.byref(p)) // 8 + 32)
        b = buf[(-buf.ctypes.data % 256) // 8:]
        fn(ctypes.byref(p), k, hc._ptrs(uk), tape.ctypes.data, dt, hc._ptrs(lam), hc._ptrs(ln), hc._ptrs(lk),
           lc.ctypes.data_as(hc._D), b.ctypes.data, int(gather))
        return ln + lk + (lc,)

    return run


@pytest.mark.parametrize("bcx", [I.PERIODIC, I.OUTFLOW])
@pytest.mark.parametrize("bcy", [I.PERIODIC, I.OUTFLOW])
@pytest.mark.parametrize("kind,nx,ny", [("smooth", 4, 4), ("smooth", 5, 9), ("shock", 12, 11), ("shock", 17, 4)])
def test_gather_is_the_scatter(oracle, points, kind, nx, ny, bcx, bcy):
    base = I.random_smooth(nx, ny, seed=3) if kind == "smooth" else I.stirred(I.random_shock(nx, ny, seed=1))
    prob = replace(base.with_size(nx, ny), bc_x=bcx, bc_y=bcy, x1=base.x0 + 1.37 * (base.x1 - base.x0))
    u0 = I.sample(prob)
    dt = oracle.dt(prob, u0)
    rng = np.random.default_rng(nx)
    lam = [rng.standard_normal(a.shape) for a in u0]
    lam[3][:, 0, :2] = 0.0
    lam[1][:, -1, :] = 0.0
    for k in (0, 1):
        _, tape = hc.record(prob, k, u0, u0, dt)
        got, ref = (points(prob, k, u0, tape, dt, tuple(lam), gather) for gather in (True, False))
        for a, b in zip(got, ref):
            for c in range(8):
                assert np.max(np.abs(a[c] - b[c])) <= BAR * (np.max(np.abs(b[c])) or 1.0)
