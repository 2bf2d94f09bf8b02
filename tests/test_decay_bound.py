"""The host's rules on the decay of T's inverse (csrc/decay_bound.hpp), compiled here and compared
with an independent evaluation of the same bounds on a fine grid, with the inverse itself, and at the
off-diagonals where the documented forms end."""
import ctypes
import math
import os
import subprocess

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
KAPPAS = [1e-12, 1e-3, 0.05, 0.25, 0.5, 0.52, 1.0, 1.1, 2.0, 4.5, 20.0, 500.0]


@pytest.fixture(scope="module")
def shipped(tmp_path_factory):
    d = tmp_path_factory.mktemp("decay")
    src, lib = d / "shim.cpp", d / "libdecay.so"
    src.write_text('#include "decay_bound.hpp"\nextern "C" {\n'
                   "int s_decoupled(double k, double b) { return decoupled(k, b); }\n"
                   "double s_halo(double k, long long s) { return window_halo(k, s); }\n"
                   "int s_levels(double k, int m) { return decay_levels(k, m, 3, 4); }\n}\n")
    subprocess.check_call(["g++", "-O1", "-std=c++17", "-shared", "-fPIC", "-o", str(lib), str(src),
                           "-I", os.path.join(ROOT, "paper_2205_00856_amd", "csrc")])
    so = ctypes.CDLL(str(lib))
    so.s_decoupled.argtypes = [ctypes.c_double, ctypes.c_double]
    so.s_halo.argtypes, so.s_halo.restype = [ctypes.c_double, ctypes.c_longlong], ctypes.c_double
    so.s_levels.argtypes = [ctypes.c_double, ctypes.c_int]
    return so


def grid(kap):
    e = np.linspace(0.0, min(8.0, math.asinh(0.5 / kap)), 400_002)[1:-1]
    return e, 2.0 * kap * np.sinh(e)


def coupling(kap, rows):
    """log2 of the best bound on two joints' coupling, kappa^2 exp(-eta (rows - 2)) / (1 - theta)."""
    e, th = grid(kap)
    return np.min(2 * np.log(kap) - e * (rows - 2) - np.log1p(-th)) / math.log(2)


@pytest.mark.parametrize("kap", KAPPAS)
def test_decoupled(shipped, kap):
    for rows in (8, 32, 64, 128, 512, 2048, 8192):
        bound = coupling(kap, rows)
        if abs(bound + 66.0) > 0.01:
            assert bool(shipped.s_decoupled(kap, rows)) == (bound <= -66.0), rows


@pytest.mark.parametrize("kap", KAPPAS)
@pytest.mark.parametrize("s", [1, 7, 50, 128])
def test_halo(shipped, kap, s):
    e, th = grid(kap)
    least = np.min((70 * math.log(2) + s * (np.log1p(th) - np.log1p(-th)) -
                    np.log(2 * np.sinh(e))) / e)
    assert least <= shipped.s_halo(kap, s) <= least * (1 + 1e-9) + 2.0


def test_documented_ends(shipped):
    """Interleaved one-pass steps up to kappa 0.56 (64 rows) and 1.20 (128), levels inside a wavefront
    up to 4.72 (8 rows per lane)."""
    assert shipped.s_decoupled(0.56, 64) and not shipped.s_decoupled(0.57, 64)
    assert shipped.s_decoupled(1.20, 128) and not shipped.s_decoupled(1.21, 128)
    assert shipped.s_levels(4.72, 8) == 6 and shipped.s_levels(4.74, 8) == -1
    levels = [shipped.s_levels(k, 8) for k in (0.1, 0.5, 1.0, 2.0, 4.0)]
    assert levels == sorted(levels) and levels[0] == 3


@pytest.mark.parametrize("kap,rows", [(0.5, 64), (1.0, 128), (4.0, 512)])
@pytest.mark.parametrize("potential", ["zero", "cancelling", "random"])
def test_joints_of_real_matrices(shipped, kap, rows, potential):
    """The coupling of two joints `rows` apart (the Schur complement's off-diagonal, formed from the
    pivots) against its diagonal, which stays at 1 or more: below 2^-66 where the rule says so."""
    g = np.random.default_rng(1)
    m = rows - 1
    v = {"zero": np.full(m, 2 * kap), "cancelling": np.zeros(m),
         "random": g.uniform(-2 * kap, 2 * kap, m)}[potential]
    assert shipped.s_decoupled(kap, rows)
    p, logc = 1 + 1j * v[0], 2 * math.log2(kap)
    for i in range(1, m):  # (T^-1)_{1,m} = prod kappa / pivots, in magnitude
        logc += math.log2(kap / abs(p))
        p = 1 + 1j * v[i] + kap * kap / p
    logc -= math.log2(abs(p))
    assert logc <= -66.0
