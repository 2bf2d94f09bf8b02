"""2^26 and more short systems: forms that number their workgroups along x alone would need 2^32
threads, which a launch does not hold; such batches take the other forms.  The systems repeat 1000
different ones, which are compared with the CPU oracle (relative L2 <= 1e-11); every system has to
equal its kind bit for bit.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("op", ["step", "propagate"])
@pytest.mark.parametrize("batch", [(1 << 24) + 77, (1 << 26) + 5])
def test_short_systems(oracle_mod, batch, op):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    n, kinds, dx, dt = 2, 1000, 0.1, 0.01
    g = np.random.default_rng(3)
    V, psi = g.uniform(-1.0, 0.0, (kinds, n)), workloads.complex_normal(g, (kinds, n))
    steps = 1 if op == "step" else 3
    ref = np.stack([oracle_mod.cn_propagate(psi[s], V[s], dx, dt, steps) for s in range(kinds)])
    rep = lambda t: torch.from_numpy(t).cuda().repeat(-(-batch // kinds), 1)[:batch].contiguous()
    tV, p = rep(V), rep(psi)
    if op == "step":
        cn.step(p, tV, dx, dt, out=p)
    else:
        cn.propagate(p, tV, dx, dt, steps)
    got = p[:kinds].clone()
    assert np.linalg.norm(got.cpu().numpy() - ref) <= 1e-11 * np.linalg.norm(ref)
    whole = batch // kinds * kinds
    assert (p[:whole].view(-1, kinds, n) == got).all()
    assert torch.equal(p[whole:], got[:batch - whole])
    assert cn.get_status() == 0
    del p, tV
    torch.cuda.empty_cache()
