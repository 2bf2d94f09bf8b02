"""GPU parity of sequences run on independent windows (k_window) against the CPU oracle stepping
one step at a time.

Tolerance: relative L2 <= 1e-11, as everywhere (FP64 on both sides; the windows' cut ends reach
their results below 2^-70 of the state).  States and potentials are random, so that every cut
would show.  Cases: one row to several windows of every size, ragged ends, off-diagonals from
far below to above 1 (the levels 3 to 6), a potential that cancels the Laplacian's diagonal,
fields, checkpoints, strided batches, one potential for a batch, and non-finite values.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-11


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


def oracle_steps(oracle_mod, psi, V, dx, dt, steps, xg=None, E=None):
    out = [psi]
    for k in range(steps):
        args = () if E is None else (xg, E[k])
        out.append(oracle_mod.cn_step(out[-1], V, dx, dt, *args))
    return out


# kappa = dt / (4 dx^2): 0.0125, 0.25, 0.5, 1, 2 and 4 (the halo of one step: 14 to 450 rows)
GRID = {0.0125: (0.4, 0.008), 0.25: (0.1, 0.01), 0.5: (0.1, 0.02), 1.0: (0.05, 0.01),
        2.0: (0.05, 0.02), 4.0: (0.03, 0.0144)}


@pytest.mark.parametrize("kap", sorted(GRID))
@pytest.mark.parametrize("n", [1, 2, 7, 9, 511, 513, 1025, 2049, 4095, 4097, 9001, 70_001])
def test_sizes_and_offdiagonals(gpu, oracle_mod, n, kap):
    torch, cn = gpu
    dx, dt = GRID[kap]
    steps = 9
    g = np.random.default_rng(n)
    V = g.uniform(-2.0, 2.0, n)
    V[n // 2:] -= 1.0 / dx ** 2  # the slowest decay: T's diagonal 1 + i tau v
    psi = workloads.complex_normal(g, n)
    xg = workloads.grid_1d(n, dx)
    E = g.normal(0.0, 0.05, steps)
    tV, tx = dev(torch, V, xg)
    for field in (False, True):
        (p,) = dev(torch, psi)
        cn.propagate(p, tV, dx, dt, steps, E=E if field else None, xgrid=tx if field else None)
        ref = oracle_steps(oracle_mod, psi, V, dx, dt, steps, xg, E if field else None)[-1]
        assert rel(p.cpu().numpy(), ref) <= TOL, field
    assert cn.get_status() == 0


@pytest.mark.parametrize("n,steps,K", [(3000, 1, 1), (20_011, 1, 4), (20_011, 2, 1),
                                       (20_011, 23, 7), (300_007, 41, 20), (2000, 300, 150)])
def test_checkpoints(gpu, oracle_mod, n, steps, K):
    """Sequences of one launch, of an odd and an even number, with states between the launches in
    the checkpoints and in the spare state; backwards in time as well (dt < 0)."""
    torch, cn = gpu
    dx, dt = 0.1, -0.02
    g = np.random.default_rng(steps)
    V = g.uniform(-2.0, 2.0, n)
    psi = workloads.complex_normal(g, n)
    ref = oracle_steps(oracle_mod, psi, V, dx, dt, steps)
    (tV,) = dev(torch, V)
    for with_ck in (False, True):
        (p,) = dev(torch, psi)
        nck = (steps + K - 1) // K
        ck = torch.zeros(nck * n, dtype=torch.complex128, device="cuda") if with_ck else None
        cn.propagate(p, tV, dx, dt, steps, ckpt=ck, K=K)
        assert rel(p.cpu().numpy(), ref[-1]) <= TOL
        if with_ck:
            c = ck.cpu().numpy().reshape(nck, n)
            for i in range(nck):
                assert rel(c[i], ref[i * K]) <= TOL, i


@pytest.mark.parametrize("n,batch,gap,shared", [(300, 5, 0, False), (700, 33, 13, False),
                                                (5000, 3, 7, False), (5000, 3, 0, True)])
def test_batches(gpu, oracle_mod, n, batch, gap, shared):
    """Batches with gaps between the systems (left untouched) and with one potential for all."""
    torch, cn = gpu
    dx, dt, steps = 0.07, 0.013, 12
    g = np.random.default_rng(batch)
    bs = n + gap
    span = (batch - 1) * bs + n
    psi = workloads.complex_normal(g, span)
    V = g.uniform(-2.0, 2.0, n if shared else span)
    L = cn.Layout(n=n, batch=batch, elem_stride=1, batch_stride=bs, shared_coefficients=shared)
    tV, p = dev(torch, V, psi)
    cn.propagate(p, tV, dx, dt, steps, layout=L)
    out = p.cpu().numpy()
    for s in range(batch):
        r = slice(s * bs, s * bs + n)
        ref = oracle_steps(oracle_mod, psi[r], V if shared else V[r], dx, dt, steps)[-1]
        assert rel(out[r], ref) <= TOL, s
        assert np.array_equal(out[s * bs + n:(s + 1) * bs], psi[s * bs + n:(s + 1) * bs])


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("where", ["psi", "V"])
def test_non_finite_line(gpu, value, where):
    """One non-finite value makes its whole line non-finite and raises the status; the other
    systems are untouched, and the next call on the same handle is clean."""
    torch, cn = gpu
    n, batch, dx, dt, steps = 20_011, 3, 0.1, 0.02, 10
    g = np.random.default_rng(3)
    V, psi = g.uniform(-2.0, 2.0, (batch, n)), workloads.complex_normal(g, (batch, n))
    tV, p = dev(torch, V, psi)
    want = p.clone()
    cn.propagate(want, tV, dx, dt, steps)
    bad_V, bad_p = tV.clone(), p.clone()
    (bad_V if where == "V" else bad_p)[1, 4321] = value
    cn.propagate(bad_p, bad_V, dx, dt, steps)
    assert cn.get_status() == 1
    assert not torch.isfinite(torch.view_as_real(bad_p[1])).any()
    assert torch.equal(bad_p[0], want[0]) and torch.equal(bad_p[2], want[2])
    cn.propagate(p, tV, dx, dt, steps)
    assert cn.get_status() == 0 and torch.equal(p, want)


@pytest.mark.parametrize("reconstruct", [False, True])
@pytest.mark.parametrize("n,kap,steps,K", [(300, 1.0, 7, 3), (1537, 0.25, 9, 9),
                                           (9001, 0.5, 12, 5), (20_011, 2.0, 13, 4),
                                           (6000, 1.0, 160, 80)])
def test_gradients(gpu, oracle_mod, n, kap, steps, K, reconstruct):
    """The reverse mode (state and gradient backwards together) against the oracle's: segments of
    one and several launches, with and without checkpoints, accumulating into dV.  g and psi are
    within rounding; dV and dE sum over the steps and rows."""
    torch, cn = gpu
    dx, dt = GRID[kap]
    rng = np.random.default_rng(n)
    V, psi = rng.uniform(-2.0, 2.0, n), workloads.complex_normal(rng, n)
    G = workloads.complex_normal(rng, n)
    xg, E = workloads.grid_1d(n, dx) / n, rng.normal(0.0, 0.05, steps)
    rg, rV, rE = oracle_mod.cn_propagate_grad(psi, V, dx, dt, steps, G, xg, E)
    tV, tx, p, g = dev(torch, V, xg, psi, G)
    nck = (steps + K - 1) // K
    ck = torch.empty(nck * n, dtype=torch.complex128, device="cuda")
    cn.propagate(p, tV, dx, dt, steps, E=E, xgrid=tx, ckpt=ck, K=K)
    start = torch.ones(n, dtype=torch.float64, device="cuda")
    dE = torch.empty(steps, dtype=torch.float64, device="cuda")
    if reconstruct:
        keep = p.clone()
        cn.propagate_adjoint_reconstruct(p, g, tV, dx, dt, steps, K, E=E, xgrid=tx, dV=start,
                                         dE=dE)
        assert torch.equal(p, keep)
    else:
        keep = ck.clone()
        cn.propagate_adjoint(ck, g, tV, dx, dt, steps, K, E=E, xgrid=tx, dV=start, dE=dE)
        assert torch.equal(ck, keep)
    assert rel(g.cpu().numpy(), rg) <= TOL
    assert rel(start.cpu().numpy() - 1.0, rV) <= TOL
    assert rel(dE.cpu().numpy(), rE) <= TOL
    assert cn.get_status() == 0
