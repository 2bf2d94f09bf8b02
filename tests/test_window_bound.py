"""The halo of the window launches, checked on the CPU: a line cut at a bond gives, the halo's
rows away from the cut, the same state after s steps as the whole line, for any real potential."""
import math

import numpy as np
import pytest

import workloads


def halo(kap, s, bits):
    """Smallest D with r^s exp(-eta D) / (2 sinh eta) <= 2^-bits over eta, r = (1 + th) / (1 - th),
    th = 2 kap sinh(eta) < 1."""
    best = math.inf
    for eta in np.linspace(0.0, min(8.0, math.asinh(0.5 / kap)), 4002)[1:-1]:
        th = 2.0 * kap * math.sinh(eta)
        best = min(best, (bits * math.log(2.0) + s * math.log((1 + th) / (1 - th)) -
                          math.log(2.0 * math.sinh(eta))) / eta)
    return math.ceil(best)


@pytest.mark.parametrize("kap,s", [(0.05, 1), (0.25, 1), (0.25, 8), (1.0, 1), (1.0, 12), (4.0, 2)])
@pytest.mark.parametrize("potential", ["zero", "cancelling", "random"])
def test_cut_stays_away(oracle_mod, kap, s, potential):
    """2^-40 instead of 2^-70, so that the bound is seen above the rounding of FP64: the error at
    the halo's distance stays below it, and far inside the halo it does not."""
    dx = 0.1
    dt = kap * 4 * dx * dx
    D = halo(kap, s, 40)
    n = 2 * D + 200
    g = np.random.default_rng(1)
    V = {"zero": np.zeros(n), "cancelling": np.full(n, -1.0 / dx ** 2),
         "random": g.uniform(-2.0 / dx ** 2, 0.0, n)}[potential]
    psi = workloads.complex_normal(g, n)
    cut = n // 2
    whole, part = psi, psi[cut:]
    for _ in range(s):
        whole = oracle_mod.cn_step(whole, V, dx, dt)
        part = oracle_mod.cn_step(part, V[cut:], dx, dt)
    err = np.abs(whole[cut:] - part)
    assert np.max(err[D:]) <= 2.0 ** -40 * np.linalg.norm(psi)
    assert np.max(err[:2]) > 1e-6  # the cut itself is felt
