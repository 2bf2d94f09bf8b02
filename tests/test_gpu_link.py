"""GPU parity of multi-tile systems solved in one pass (k_tile<PH_LINK>) and of the tiles that such
a pass leaves to the launches after it, against the CPU oracle.

Tolerance: relative L2 <= 1e-11, as everywhere (the couplings that a tile drops are below 2^-66 of
its diagonal); for steps with a large kappa 16 * 4 kappa * 2^-53, the rounding of a matrix of norm
1 + 4 kappa whose inverse has norm 1.  Ill-conditioned matrices (slow, mixed: condition 2e7) are
compared with the two-pass form on the same tiles (an explicit partition): bit for bit where every
joint couples, else to 1e-11.  The plans take one pass from 2^20 rows on.  Cases: matrices whose joints decouple,
matrices whose do not (the whole system in two passes), both kinds in one system, ragged ends, in
place and out of place, the conjugate transpose, batches, uneven batches with a spacing per
system, absorbing potentials, several calls in a row, graph replays, and non-finite values.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-11
N = (1 << 20) + 777


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


def dev(torch, *arrs):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrs]


def system(n, kind, seed=1):
    """a, b, c, d: fast (diagonally dominant, couplings 1/4), slow (the joints of neighbouring
    tiles couple: off-diagonals 1 - 1e-7 of half the diagonal) or half slow rows, half fast."""
    g = np.random.default_rng(seed)
    slow = {"fast": np.zeros(n, bool), "slow": np.ones(n, bool),
            "mixed": (np.arange(n) // 100_000) % 2 == 0}[kind]
    a = 2.0 + 0.1j * g.standard_normal(n) * ~slow
    off = np.where(slow, -(1.0 - 1e-7), 0.25)
    b, c = off * np.exp(0.3j * ~slow), off * np.exp(-0.2j * ~slow)
    return a, b + 0j, c + 0j, workloads.complex_normal(g, n)


def check(torch, cn, oracle_mod, kind, mats, got):
    a, b, c, d = mats
    if kind == "fast":
        assert rel(got.cpu().numpy(), oracle_mod.thomas(a, b, c, d)) <= TOL
        return
    two = cn.solve(*dev(torch, a, b, c, d),
                   layout=cn.Layout.contiguous(len(d), 1, partition=1024, rows_per_thread=4))
    if kind == "slow":
        assert torch.equal(got, two)
    assert rel(got.cpu().numpy(), two.cpu().numpy()) <= TOL


@pytest.mark.parametrize("n", [N, 1 << 21])
@pytest.mark.parametrize("kind", ["fast", "slow", "mixed"])
def test_solve(gpu, oracle_mod, kind, n):
    torch, cn = gpu
    a, b, c, d = system(n, kind)
    ta, tb, tc, td = dev(torch, a, b, c, d)
    assert "one pass" in cn.describe_plan(cn.Layout.contiguous(n, 1))
    x = cn.solve(ta, tb, tc, td)
    check(torch, cn, oracle_mod, kind, (a, b, c, d), x)
    for _ in range(3):  # in place, the two line buffers in turn, the same bits
        y = td.clone()
        cn.solve(ta, tb, tc, y, out=y)
        assert torch.equal(x, y)
    assert cn.get_status() == 0


def test_alternating_kinds(gpu, oracle_mod):
    """Calls that finish in one pass and calls that do not, on one plan."""
    torch, cn = gpu
    for s, kind in enumerate(["fast", "slow", "slow", "fast", "mixed", "fast"]):
        mats = system(N, kind, s)
        check(torch, cn, oracle_mod, kind, mats, cn.solve(*dev(torch, *mats)))


@pytest.mark.parametrize("kind", ["fast", "mixed"])
def test_transposed(gpu, oracle_mod, kind):
    torch, cn = gpu
    a, b, c, d = system(N, kind)
    if kind == "fast":
        x = oracle_mod.thomas(a, b, c, d)
        want = oracle_mod.thomas_adjoint(a, b, c, x, d)
    else:
        x = d
        L = cn.Layout.contiguous(N, 1, partition=1024, rows_per_thread=4)
        want = [t.cpu().numpy() for t in cn.solve_adjoint(*dev(torch, a, b, c, x, d), layout=L)]
    got = cn.solve_adjoint(*dev(torch, a, b, c, x, d))
    for t, ref in zip(got, want):
        assert rel(t.cpu().numpy(), ref) <= TOL


@pytest.mark.parametrize("absorb", [False, True])
@pytest.mark.parametrize("kap", [0.5, 50.0, 5e5])
def test_step(gpu, oracle_mod, kap, absorb):
    """Steps in place (edge rows next to stored ones), joints that decouple and (5e5) not."""
    torch, cn = gpu
    dt = 0.02
    dx = 0.5 * np.sqrt(dt / kap)
    g = np.random.default_rng(7)
    V, psi = g.uniform(-1.0, 0.0, N), workloads.complex_normal(g, N)
    W = workloads.absorber(N) if absorb else None
    ref = psi
    tV, p = dev(torch, V, psi)
    tW = dev(torch, W)[0] if absorb else None
    for _ in range(3):
        ref = oracle_mod.cn_step(ref, V, dx, dt, W=W)
        cn.step(p, tV, dx, dt, out=p, W=tW)
    tol = max(TOL, 64 * kap * 2.0 ** -53)
    assert rel(p.cpu().numpy(), ref) <= 3 * tol
    out = cn.step(dev(torch, psi)[0], tV, dx, dt, W=tW)
    assert rel(out.cpu().numpy(), oracle_mod.cn_step(psi, V, dx, dt, W=W)) <= tol


@pytest.mark.parametrize("n,batch,linked", [((1 << 18) - 2048, 1, False),
                                            ((1 << 18) - 2047, 1, True), (1 << 15, 8, True),
                                            ((1 << 15) - 1, 8, False), (400_003, 1, True)])
def test_absorbing_sequences(gpu, oracle_mod, n, batch, linked):
    """Absorbing steps on both sides of the rule that takes them in one pass: chained steps
    (propagate) and single ones against the oracle, which steps system by system."""
    torch, cn = gpu
    dx, dt, steps = 0.1, 0.012, 3
    g = np.random.default_rng(n)
    V, W = g.uniform(-1.0, 0.0, n * batch), g.uniform(0.0, 1.0, n * batch)
    psi = workloads.complex_normal(g, n * batch)
    L = cn.Layout.contiguous(n, batch)
    assert ("one pass over the tiles" in cn.describe_plan(L, absorbing=True)) == linked
    tV, tW, p, q = dev(torch, V, W, psi, psi)
    cn.propagate(p, tV, dx, dt, steps, W=tW, layout=L)
    for _ in range(steps):
        cn.step(q, tV, dx, dt, out=q, W=tW, layout=L)
    ref = np.concatenate([oracle_mod.cn_propagate(psi[i * n:(i + 1) * n], V[i * n:(i + 1) * n], dx,
                                                  dt, steps, W=W[i * n:(i + 1) * n])
                          for i in range(batch)])
    assert rel(p.cpu().numpy(), ref) <= TOL
    assert rel(q.cpu().numpy(), ref) <= TOL


def test_batches(gpu, oracle_mod):
    """A uniform batch of several tiles each, and an uneven one with a spacing per system (some
    systems coupled, some not)."""
    torch, cn = gpu
    n, batch, dt = 9001, 150, 0.02
    g = np.random.default_rng(5)
    V, psi = g.uniform(-1.0, 0.0, (batch, n)), workloads.complex_normal(g, (batch, n))
    tV, p = dev(torch, V, psi)
    cn.step(p, tV, 0.1, dt, out=p)
    out = p.cpu().numpy()
    for s in range(0, batch, 29):
        assert rel(out[s], oracle_mod.cn_step(psi[s], V[s], 0.1, dt)) <= TOL
    lens = np.concatenate([[1, 4097, 2048, 65_536], g.integers(3000, 20_000, 120)])
    offs = np.concatenate([[0], np.cumsum(lens)])
    dx = np.where(np.arange(len(lens)) % 7 == 3, 1e-4, g.uniform(0.05, 0.2, len(lens)))
    V, psi = g.uniform(-1.0, 0.0, offs[-1]), workloads.complex_normal(g, offs[-1])
    tV, p, tdx = dev(torch, V, psi, dx)
    L = cn.Layout.uneven(offs)
    assert "one pass" in cn.describe_plan(L, cn_mode=True)
    for _ in range(2):
        cn.step(p, tV, 0.0, dt, dx_per_system=tdx, out=p, layout=L)
    out = p.cpu().numpy()
    for s in range(len(lens)):
        r = slice(offs[s], offs[s + 1])
        ref = oracle_mod.cn_step(psi[r], V[r], dx[s], dt)
        tol = max(TOL, 2 * 64 * dt / (4 * dx[s] ** 2) * 2.0 ** -53)
        assert rel(out[r], oracle_mod.cn_step(ref, V[r], dx[s], dt)) <= tol, s


def test_graph_replays(gpu):
    torch, cn = gpu
    a, b, c, d = dev(torch, *system(N, "mixed"))
    want = cn.solve(a, b, c, d)
    x = d.clone()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cn.solve(a, b, c, x, out=x)
    for _ in range(3):
        x.copy_(d)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(x, want)
        assert torch.equal(cn.solve(a, b, c, d), want)  # eager work between the replays


def test_non_finite(gpu):
    """One NaN makes its whole system NaN and raises the status; other systems of the batch and
    the next call are clean."""
    torch, cn = gpu
    n, batch = 300_001, 4
    mats = [system(n, "fast", s) for s in range(batch)]
    a, b, c, d = (torch.stack(t) for t in zip(*(dev(torch, *m) for m in mats)))
    L = cn.Layout.contiguous(n, batch)
    want = cn.solve(a, b, c, d, layout=L)
    bad = d.clone()
    bad[2, 123_456] = float("nan")
    x = cn.solve(a, b, c, bad, out=bad, layout=L)
    assert cn.get_status() == 1
    assert not torch.isfinite(torch.view_as_real(x[2])).any()
    for s in (0, 1, 3):
        assert torch.equal(x[s], want[s])
    assert torch.equal(cn.solve(a, b, c, d, layout=L), want)
    assert cn.get_status() == 0


@pytest.mark.parametrize("n,batch", [(N, 1 + 15), (1 << 20, 2), (N, 5)])
@pytest.mark.parametrize("kind", ["fast", "slow", "mixed"])
def test_several_right_hand_sides(gpu, oracle_mod, kind, n, batch):
    """One matrix with an even and an odd number of right-hand sides, in place."""
    torch, cn = gpu
    a, b, c, _ = system(n, kind)
    d = np.stack([system(n, "fast", s)[3] for s in range(batch)])
    ta, tb, tc, td = dev(torch, a, b, c, d)
    L = cn.Layout.contiguous(n, batch, shared_coefficients=True)
    assert "one pass" in cn.describe_plan(L) and "rhs/wg=" in cn.describe_plan(L)
    x = cn.solve(ta, tb, tc, td, layout=L)
    for s in {0, batch // 2, batch - 1}:
        check(torch, cn, oracle_mod, kind, (a, b, c, d[s]), x[s])
    for _ in range(2):
        y = td.clone()
        cn.solve(ta, tb, tc, y, out=y, layout=L)
        assert torch.equal(x, y)
    bad = td.clone()
    bad[batch - 1, n // 2] = float("inf")
    cn.get_status() if kind == "fast" else None
    cn.solve(ta, tb, tc, bad, out=bad, layout=L)
    assert cn.get_status() == 1
    assert not torch.isfinite(torch.view_as_real(bad[batch - 1])).any()
    assert torch.equal(bad[:-1], x[:-1])
    assert torch.equal(cn.solve(ta, tb, tc, td, layout=L), x)
    assert cn.get_status() == 0


@pytest.mark.parametrize("n,batch", [(1025, 3), (2048, 1), (65_536, 1), (100_003, 2), (9001, 40)])
@pytest.mark.parametrize("shared", [False, True])
def test_smaller_solves(gpu, oracle_mod, n, batch, shared):
    """512-row tiles (from 2^16 rows on) and whole systems of 1025 to 2048 rows, forward and
    transposed, one matrix each and one for all."""
    torch, cn = gpu
    mats = [system(n, "fast", s) for s in range(1 if shared else batch)]
    d = np.stack([system(n, "fast", 50 + s)[3] for s in range(batch)])
    a, b, c = (torch.stack(dev(torch, *t)) for t in list(zip(*mats))[:3])
    (td,) = dev(torch, d)
    L = cn.Layout.contiguous(n, batch, shared_coefficients=shared)
    x = cn.solve(a, b, c, td, layout=L)
    for s in range(batch):
        m = mats[0 if shared else s]
        assert rel(x[s].cpu().numpy(), oracle_mod.thomas(*m[:3], d[s])) <= TOL
    if not shared:
        lam = cn.solve_adjoint(a, b, c, x, td, need_abc=False, layout=L)[0].cpu().numpy()
        for s in range(batch):
            ref = oracle_mod.thomas_adjoint(*mats[s][:3], x[s].cpu().numpy(), d[s])[0]
            assert rel(lam[s], ref) <= TOL
    assert cn.get_status() == 0
