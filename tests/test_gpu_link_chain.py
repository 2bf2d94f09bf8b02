"""Sequences over tiles whose joints couple: once a pass has reported a left tile, the next sequence
is chained (no launch of single steps is logged) instead of two passes a step, and its result is
that of single steps within rounding: 16 * 4 kappa * 2^-53 per step, the rounding of a matrix of norm
1 + 4 kappa whose inverse has norm 1."""
import pytest

pytestmark = pytest.mark.gpu


def test_chained_where_joints_couple():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    n, dx, dt, steps = (1 << 21) + 4099, 0.01, 0.1, 6
    kap = dt / 4 / dx ** 2
    g = torch.Generator(device="cuda").manual_seed(2)
    V = torch.full((n,), -1.0 / dx ** 2, dtype=torch.float64, device="cuda")
    psi = torch.randn(n, dtype=torch.complex128, device="cuda", generator=g)
    one = psi.clone()
    for _ in range(steps):
        cn.step(one, V, dx, dt, out=one)
        torch.cuda.synchronize()
    cn.profile(True)
    try:
        seq = psi.clone()
        cn.propagate(seq, V, dx, dt, steps)
        torch.cuda.synchronize()
        logged = cn.profile_report()
    finally:
        cn.profile(False)
    assert logged == []
    assert ((seq - one).norm() / one.norm()).item() <= steps * 16 * 4 * kap * 2.0 ** -53
    assert cn.get_status() == 0


def test_description_names_the_forms_of_a_sequence():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    def forms(L, **kw):
        d = cn.describe_plan(L, **kw)
        return ["windows" in d, "single one-pass steps" in d, "chain: one fused pass" in d]

    n = (1 << 20) + 5
    assert forms(cn.Layout.contiguous(n, 1), cn_mode=True) == [True, True, True]
    assert forms(cn.Layout.contiguous(n, 1), absorbing=True) == [False, True, True]
    assert forms(cn.Layout.contiguous(n, 1, partition=2048), cn_mode=True) == [False, False, True]
    assert forms(cn.Layout.contiguous(300, 64), cn_mode=True) == [True, False, False]
    assert forms(cn.Layout.interleaved(300, 64), cn_mode=True) == [False, False, False]
