"""Rounding errors of the one-pass steps and of the sequences on windows: measured against 80-bit
arithmetic (the coefficients rounded to FP64 first, as every form rounds them), over 64 systems at
once they are those of plain FP64 half-steps and eliminations in the textbook order.  The bound, 1.2
times the latter, allows for another order of elimination; forms with fewer operations (T y = psi and
psi' = 2 y - psi, rows divided by kappa) leave 1.3 to 4 times as much.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
N, B, STEPS = 300, 64, 40


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    cn.handle(0)
    return torch, cn


def steps(psi, V, x, E, dx, dt, real, cplx):
    """Crank-Nicolson steps of B systems at once, row by row: explicit half, then Thomas."""
    tau, idx2 = 0.5 * dt, 1.0 / (dx * dx)
    kap = real(0.5 * tau * idx2)
    off = cplx(-1j) * kap
    psi = psi.astype(cplx)
    for e in E:
        v = (tau * (idx2 + (V + x * e))).astype(real)  # FP64 coefficients in either arithmetic
        s = np.zeros_like(psi)
        s[:, 1:] += psi[:, :-1]
        s[:, :-1] += psi[:, 1:]
        d = psi - cplx(1j) * v * psi + cplx(1j) * kap * s
        a = cplx(1) + cplx(1j) * v
        c = np.empty_like(psi)
        for i in range(N):
            p, q = a[:, i], d[:, i]
            if i:
                p, q = p - off * c[:, i - 1], q - off * psi[:, i - 1]
            r = cplx(1) / p
            c[:, i], psi[:, i] = off * r, q * r
        for i in range(N - 2, -1, -1):
            psi[:, i] -= c[:, i] * psi[:, i + 1]
    return psi


@pytest.fixture(scope="module")
def cases():
    made = {}

    def get(dx, dt, field, state):
        k = (dx, dt, field, state)
        if k not in made:
            g = np.random.default_rng(int(1e4 * dx) + field)
            x = np.broadcast_to((np.arange(N) - N / 2) * dx, (B, N)).copy()
            V = -1.0 / np.sqrt((x - g.uniform(-1, 1, (B, 1))) ** 2 + 2.0)
            psi = (workloads.complex_normal(g, (B, N)) if state == "rough" else
                   np.exp(-(x - g.uniform(-1, 1, (B, 1))) ** 2 / 8 + 1j * g.uniform(.5, 1.5, (B, 1)) * x))
            E = (0.05 * g.standard_normal(STEPS)) if field else np.zeros(STEPS)
            true = steps(psi, V, x, E, dx, dt, np.longdouble, np.clongdouble)
            plain = steps(psi, V, x, E, dx, dt, np.float64, np.complex128)
            made[k] = psi, V, x, E, true, float(np.linalg.norm(plain - true) / np.linalg.norm(true))
        return made[k]

    return get


# kappa 0.25, 0.5, 1.0 and 0.33
@pytest.mark.parametrize("dx,dt", [(0.1, 0.01), (0.1, 0.02), (0.05, 0.01), (0.0862, 0.0098)])
@pytest.mark.parametrize("field", [False, True])
@pytest.mark.parametrize("state", ["rough", "packet"])
@pytest.mark.parametrize("form", ["rows", "columns", "windows"])
def test_rounding(gpu, cases, form, state, field, dx, dt):
    torch, cn = gpu
    psi, V, x, E, true, plain = cases(dx, dt, field, state)
    dev = lambda t: torch.from_numpy(np.ascontiguousarray(t.T if form == "columns" else t)).cuda()
    p, tV, tx = dev(psi), dev(V), dev(x)
    if form == "windows":
        cn.propagate(p, tV, dx, dt, STEPS, **(dict(E=E, xgrid=tx) if field else {}))
    else:
        L = cn.Layout.interleaved(N, B) if form == "columns" else cn.Layout.contiguous(N, B)
        for e in E:
            cn.step(p, tV, dx, dt, out=p, layout=L, **(dict(E=float(e), xgrid=tx) if field else {}))
    got = p.cpu().numpy()
    got = got.T if form == "columns" else got
    err = float(np.linalg.norm(got - true) / np.linalg.norm(true))
    assert err <= 1.2 * plain, (err, plain)
