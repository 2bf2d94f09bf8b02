"""Checkpoints of a sequence on windows when a state is not finite: as in single steps, every state
after the first step of such a system is non-finite in all of its rows, and so are the gradients."""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("value", [np.nan, np.inf])
@pytest.mark.parametrize("resident", [False, True])
def test_checkpoints_of_a_non_finite_line(value, resident):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    n, batch, dx, dt, steps, K = 20_011, 1 if resident else 3, 0.1, 0.02, 11, 3
    g = np.random.default_rng(4)
    V, psi = g.uniform(-2.0, 2.0, (batch, n)), workloads.complex_normal(g, (batch, n))
    tV, p0 = torch.from_numpy(V).cuda(), torch.from_numpy(psi).cuda()
    nck = -(-steps // K)
    call = cn.propagate_resident if resident else cn.propagate
    if resident:
        tV, p0 = tV[0].contiguous(), p0[0].contiguous()

    def run(p):
        ck = torch.empty(nck * batch * n, dtype=torch.complex128, device="cuda")
        call(p, tV, dx, dt, steps, ckpt=ck, K=K)
        return ck.view(nck, batch, n)

    want = run(p0.clone())
    bad = p0.clone()
    s = batch // 2
    bad.view(batch, n)[s, 4321] = value
    keep = bad.clone().view(batch, n)
    ck = run(bad)
    assert cn.get_status() == 1
    fin = torch.isfinite(torch.view_as_real(ck)).all(-1)
    assert not fin[1:, s].any()
    assert fin[0, s].sum() == n - 1 and torch.equal(ck[0, s, :4321], keep[s, :4321])
    for other in range(batch):
        if other != s:
            assert torch.equal(ck[:, other], want[:, other])
    assert torch.equal(run(p0.clone()), want)
    assert cn.get_status() == 0
    if not resident:
        G = torch.from_numpy(workloads.complex_normal(g, (batch, n))).cuda()
        dV = torch.zeros_like(tV)
        cn.propagate_adjoint(ck, G, tV, dx, dt, steps, K, dV=dV,
                             layout=cn.Layout.contiguous(n, batch))
        assert cn.get_status() == 1
        assert torch.isnan(dV[s]).all()
        assert all(torch.isfinite(dV[o]).all() for o in range(batch) if o != s)


@pytest.mark.parametrize("n", [300, 20_011])
def test_no_checkpoints_any_interval(n):
    """Without checkpoints their interval has no meaning and may be 0."""
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    g = np.random.default_rng(5)
    V = torch.from_numpy(g.uniform(-2.0, 2.0, n)).cuda()
    p = torch.from_numpy(workloads.complex_normal(g, n)).cuda()
    want = cn.propagate(p.clone(), V, 0.1, 0.02, 7).clone()
    assert torch.equal(cn.propagate(p.clone(), V, 0.1, 0.02, 7, K=0), want)
    assert torch.equal(cn.propagate_resident(p.clone(), V, 0.1, 0.02, 7, K=0), want)
