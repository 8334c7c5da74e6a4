"""Step (2) of the flux limiter as the FP64 cell tile runs it (sixteen lanes a
cell), built for the host, against the oracle bit for bit: Lambda, root solves,
fallbacks.  The boxes are the committed jets-like ones and boxes whose energy
drop empties a vertex's pressure to round-off: there a vertex asks for a root
and the cubic, which rounds differently, returns 1, so that only the check of
the final box keeps the vertex in G."""
import ctypes
import os
import subprocess
import sys

import numpy as np
import pytest

from limiter_cases import G, box_cases, in_G, low_beta, p_of
from paper_2506_04857_amd.inputs import prim_to_cons

sys.path.insert(0, os.path.dirname(os.path.abspath(__file__)))
from hostcheck import hostcheck as hc  # noqa: E402

COUNTERS = ("n_llf_not_admissible", "n_newton", "newton_iters_max", "n_fallback")


def emptied_cases(seed=2506 + 75, count=600):
    """Boxes with one to four interfaces that lower the energy alone, together
    to a pressure of zero up to round-off."""
    rng = np.random.default_rng(seed)
    out = []
    for n in range(count):
        A1 = prim_to_cons(low_beta(rng, 1e-8, 1e-2), G)
        if not in_G(A1):
            continue
        H = np.zeros((4, 8))
        w = rng.random(4) * (rng.random(4) < 0.6)
        w[n % 4] += 0.1
        H[:, 7] = -w / w.sum() * p_of(A1) / (G - 1)
        out.append((A1, H, min(1e-13, A1[0]), min(1e-13, p_of(A1))))
    return out


@pytest.fixture(scope="module")
def box_lanes(tmp_path_factory):
    out = str(tmp_path_factory.mktemp("box") / "libbox.so")
    subprocess.check_call(["g++", "-O2", "-std=c++20", "-ffp-contract=off", "-fPIC", "-shared", "-pthread", "-w",
                           "-I", os.path.join(hc.HERE, "device_stub"), "-I", hc.CSRC,
                           os.path.join(hc.HERE, "box_lanes_check.cpp"), "-o", out])
    fn = ctypes.CDLL(out).hc_box_lanes
    fn.argtypes = [ctypes.c_long, ctypes.c_double, hc._D, hc._D, ctypes.POINTER(ctypes.c_ulonglong)]
    fn.restype = None

    def run(cases):
        x = np.array([np.concatenate([a1, H.ravel(), [er, ep]]) for a1, H, er, ep in cases])
        lam, cnt = np.empty((len(cases), 4)), np.zeros(10, dtype=np.uint64)
        fn(len(cases), G, x.ctypes.data_as(hc._D), lam.ctypes.data_as(hc._D),
           cnt.ctypes.data_as(ctypes.POINTER(ctypes.c_ulonglong)))
        return lam, dict(zip(COUNTERS, cnt.tolist()))

    return run


@pytest.mark.parametrize("kind", ["jets", "emptied"])
def test_box_lanes_bitwise(oracle, box_lanes, kind):
    cases = box_cases(count=600) if kind == "jets" else emptied_cases()
    got, cnt = box_lanes(cases)
    nn = nf = 0
    whole = 0  # boxes whose roots are all exactly 1
    for (a1, H, er, ep), g in zip(cases, got):
        lam, info = oracle.flux_limiter_box(a1, H, G, er, ep)
        nn += info["n_newton"]
        nf += info["n_fallback"]
        whole += info["n_fallback"] > 0 and np.all(info["lambda_before_fallback"] == 1.0)
        np.testing.assert_array_equal(g, lam)
    assert cnt["n_newton"] == nn and cnt["n_fallback"] == nf and nf > 20
    assert kind == "jets" or whole > 20
