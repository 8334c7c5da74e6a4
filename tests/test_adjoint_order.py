"""A stage's reverse sums the contributions of points and cells in an order that
the launches, and on the GPU the atomic additions, decide.  The gradient of
limited data may not depend on it.  Where a centre value's density is limited to
1e-13, the pressure's derivative with respect to that density is large, so that
a contribution which cancels in exact arithmetic would turn the last bits of what
was summed before into 1e-9 to 1e-6 of the gradient.

A step's gradient on the host, points first and cells first.  The bar is that of the other
comparison of two orders of summation (test_adjoint_gather.py), 1e-11 of each
component's largest entry."""
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
def points_first(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("order") / "liborder.so")
    subprocess.check_call(["g++", "-O2", "-std=c++17", "-ffp-contract=off", "-fPIC", "-shared", "-I", hc.CSRC,
                           os.path.join(hc.HERE, "adjoint_order_check.cpp"), "-o", out])
    fn = ctypes.CDLL(out).hc_adjoint_points_first
    fn.argtypes = hc.lib().hc_adjoint.argtypes
    fn.restype = None

    def run(prob, k, uk, tape, dt, lam, ln, lk):
        p = hc._params(prob)
        buf = np.zeros(hc.lib().hc_adjbuf_bytes(ctypes.byref(p)) // 8 + 32)
        b = buf[(-buf.ctypes.data % 256) // 8:]
        fn(ctypes.byref(p), k, hc._ptrs(uk), tape.ctypes.data, dt, hc._ptrs(lam), hc._ptrs(ln), hc._ptrs(lk),
           b.ctypes.data)

    return run


def density_limited(prob, u):
    """Cells whose unlimited centre value has a density below the bound."""
    a, x, y, v = (t[0] for t in u)
    nxt = lambda t, ax: np.roll(t, -1, ax) if t.shape[ax] == a.shape[ax] else np.delete(t, 0, ax)  # noqa: E731
    cut = lambda t: t[:prob.ny, :prob.nx]  # noqa: E731
    faces = cut(x) + cut(nxt(x, 1)) + cut(y) + cut(nxt(y, 0))
    corners = cut(v) + cut(nxt(v, 1)) + cut(nxt(v, 0)) + cut(nxt(nxt(v, 0), 1))
    return int(np.sum((36 * a - 4 * faces - corners) / 16 < 1e-13))


def calm(base):
    """base with its velocities 0 (stirred() adds small ones: near rest the
    pressure's derivative outweighs the rest the most)."""
    def prim(x, y, t):
        w = np.array(base.prim(x, y, t) * np.ones_like(np.asarray(x, dtype=np.float64)))
        w[1:4] = 0.0
        return w

    return replace(base, prim=prim)


@pytest.mark.parametrize("bc", [I.OUTFLOW, I.PERIODIC])
@pytest.mark.parametrize("nx,ny,seed", [(24, 18, 0), (24, 18, 3), (24, 18, 5), (40, 40, 2)])
def test_order_of_addition(oracle, points_first, nx, ny, bc, seed):
    prob = I.stirred(calm(I.random_shock(nx, ny, seed=seed, bc=bc)))
    u = I.sample(prob)
    assert density_limited(prob, u) > 0
    dt = oracle.dt(prob, u)
    u1, t0 = hc.record(prob, 0, u, u, dt)
    u2, t1 = hc.record(prob, 1, u, u1, dt)
    _, t2 = hc.record(prob, 2, u, u2, dt)
    grads = []
    for reverse in (hc.adjoint, points_first):
        lam = tuple(np.random.default_rng(seed).standard_normal(a.shape) for a in u)
        ln, l2, l1 = (tuple(np.zeros_like(a) for a in u) for _ in range(3))
        reverse(prob, 2, u2, t2, dt, lam, ln, l2)
        reverse(prob, 1, u1, t1, dt, l2, ln, l1)
        reverse(prob, 0, u, t0, dt, l1, ln, ln)
        grads.append(ln)
    for a, b in zip(*grads):
        for c in range(8):
            assert np.max(np.abs(a[c] - b[c])) <= BAR * np.max(np.abs(b[c]))
