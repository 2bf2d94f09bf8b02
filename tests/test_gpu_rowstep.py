"""GPU parity of the one-pass step of contiguous systems (k_rowstep) and of the real form of the
partial waves' field part (k_lstep) against the CPU oracle.  Tolerance: relative L2 <= 1e-11 per
system, as everywhere (joints are taken as decoupled below 2^-66).  Cases: every tile that holds a
whole system, at and around its edges, systems of several tiles, the levels 3 to 6, the slowest
decay, a field, one potential for a batch, gaps, in place and out of place, captured calls, and
non-finite values.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-11
GRID = {0.02: (0.5, 0.02), 0.5: (0.1, 0.02), 1.0: (0.05, 0.01), 2.0: (0.05, 0.02),
        4.0: (0.03, 0.0144)}


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    cn.handle(0)
    return torch, cn


def rel(x, y):
    return float(np.linalg.norm(x - y) / max(np.linalg.norm(y), 1e-300))


@pytest.mark.parametrize("kap", sorted(GRID))
@pytest.mark.parametrize("n", [1, 2, 9, 256, 257, 384, 385, 512, 513, 768, 1024, 1025, 1537, 2049,
                               3073, 4096, 4097, 6144, 20_011])
def test_step(gpu, oracle_mod, n, kap):
    torch, cn = gpu
    dx, dt = GRID[kap]
    g = np.random.default_rng(n)
    batch, bs = 3, n + n % 5
    span = (batch - 1) * bs + n
    V, psi = g.uniform(-2.0, 2.0, span), workloads.complex_normal(g, span)
    V[span // 2:] -= 1.0 / dx ** 2
    x = g.uniform(-3.0, 3.0, span)
    L = cn.Layout(n=n, batch=batch, elem_stride=1, batch_stride=bs)
    tV, tx, p0 = (torch.from_numpy(t).cuda() for t in (V, x, psi))
    for E in (0.0, 0.3):
        kw = dict(E=E, xgrid=tx) if E else {}
        out = torch.full_like(p0, 7.0)
        cn.step(p0, tV, dx, dt, v_scale=0.5, out=out, layout=L, **kw)
        inp = p0.clone()
        cn.step(inp, tV, dx, dt, v_scale=0.5, out=inp, layout=L, **kw)
        a, b = out.cpu().numpy(), inp.cpu().numpy()
        for s in range(batch):
            r = slice(s * bs, s * bs + n)
            args = (x[r], E) if E else ()
            ref = oracle_mod.cn_step(psi[r], 0.5 * V[r], dx, dt, *args)
            assert rel(a[r], ref) <= TOL and rel(b[r], ref) <= TOL, (s, E)
        assert (a[n:bs] == 7.0).all() and (b[n:bs] == psi[n:bs]).all()
    assert cn.get_status() == 0


def test_shared_potential(gpu, oracle_mod):
    torch, cn = gpu
    n, batch, dx, dt = 5000, 4, 0.1, 0.02
    g = np.random.default_rng(2)
    V, psi = g.uniform(-2.0, 2.0, n), workloads.complex_normal(g, (batch, n))
    L = cn.Layout.contiguous(n, batch, shared_coefficients=True)
    out = cn.step(torch.from_numpy(psi).cuda(), torch.from_numpy(V).cuda(), dx, dt, layout=L)
    for s in range(batch):
        assert rel(out[s].cpu().numpy(), oracle_mod.cn_step(psi[s], V, dx, dt)) <= TOL


def test_repeated_and_captured(gpu):
    torch, cn = gpu
    n, dx, dt = 100_003, 0.1, 0.02
    g = np.random.default_rng(4)
    tV = torch.from_numpy(g.uniform(-2.0, 2.0, n)).cuda()
    p0 = torch.from_numpy(workloads.complex_normal(g, n)).cuda()

    def steps(p):
        for _ in range(3):
            cn.step(p, tV, dx, dt, out=p)
        return p

    want = steps(p0.clone())
    assert torch.equal(steps(p0.clone()), want)
    p = p0.clone()
    gr = torch.cuda.CUDAGraph()
    with torch.cuda.graph(gr):
        steps(p)
    for _ in range(3):
        p.copy_(p0)
        torch.cuda.synchronize()
        gr.replay()
        torch.cuda.synchronize()
        assert torch.equal(p, want)
        assert torch.equal(steps(p0.clone()), want)  # eager work between the replays


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("where", ["psi", "V"])
@pytest.mark.parametrize("n", [400, 3000, 20_011])
def test_non_finite_system(gpu, n, value, where):
    """One non-finite value makes its whole system NaN and raises the status; the other systems
    and the next call are clean."""
    torch, cn = gpu
    g = np.random.default_rng(3)
    dx, dt = 0.1, 0.02
    tV = torch.from_numpy(g.uniform(-2.0, 2.0, (3, n))).cuda()
    p0 = torch.from_numpy(workloads.complex_normal(g, (3, n))).cuda()
    want = cn.step(p0, tV, dx, dt)
    bV, bp = tV.clone(), p0.clone()
    (bV if where == "V" else bp)[1, n // 3] = value
    cn.step(bp, bV, dx, dt, out=bp)
    assert cn.get_status() == 1
    assert not torch.isfinite(torch.view_as_real(bp[1])).any()
    assert torch.equal(bp[0], want[0]) and torch.equal(bp[2], want[2])
    assert torch.equal(cn.step(p0, tV, dx, dt), want)
    assert cn.get_status() == 0


@pytest.mark.parametrize("nr,nl,l0,E", [(64, 1, 0, 0.3), (65, 8, 0, 0.3), (1000, 9, 2, -0.4),
                                        (129, 63, 0, 2.0), (5000, 64, 1, 0.1), (300, 65, 0, 0.2)])
def test_partial_waves(gpu, oracle_mod, nr, nl, l0, E):
    """Radial part with the centrifugal potential formed in the kernel, field part as a real system
    (65 waves: the complex column kernels); in place."""
    torch, cn = gpu
    dr, dt = 0.1, 0.02
    g = np.random.default_rng(nr)
    r = np.arange(1, nr + 1) * dr
    V, psi = -1.0 / np.sqrt(r * r + 0.5), workloads.complex_normal(g, nl * nr)
    tV, p = torch.from_numpy(V).cuda(), torch.from_numpy(psi).cuda()
    ref = oracle_mod.radial_step(psi, V, dr, dt, E, l0, nl)
    cn.radial_step(p, tV, dr, dt, E, l0, nl, out=p)
    assert rel(p.cpu().numpy(), ref) <= TOL
    assert cn.get_status() == 0
