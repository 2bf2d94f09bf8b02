"""Tiles that a one-pass form leaves to the launch after it.  CN_LINK_SPIN=0 makes every wait for a
neighbour's line give up before its first poll, so all tiles are left; 1 leaves those whose
neighbours are late, beside tiles that are stored.  Either way the results are those of an ordinary
pass bit for bit, in place and out of place, and a non-finite value makes its whole system NaN.
Every case has a layout of its own: a plan of linked tiles that left one goes back to two passes.
"""
import itertools

import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
OPS = ["solve", "adjoint", "mrhs", "absorbing", "uneven", "rows", "columns", "columns128"]
CASES = list(itertools.product(OPS, [0, 1], [False, True], [False, True]))


def same(torch, a, b):
    a, b = (torch.view_as_real(t) for t in (a, b))
    return torch.equal(torch.isnan(a), torch.isnan(b)) and torch.equal(
        torch.nan_to_num(a), torch.nan_to_num(b))


@pytest.mark.parametrize("op,spin,inplace,nan", CASES)
def test_left_tiles(monkeypatch, op, spin, inplace, nan):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    k = CASES.index((op, spin, inplace, nan))
    g = np.random.default_rng(k)
    dev = lambda t: torch.from_numpy(np.ascontiguousarray(t)).cuda()
    normal = lambda *shape: dev(workloads.complex_normal(g, shape))
    if op in ("solve", "adjoint", "mrhs"):
        n, rhs = (1 << 17) + 37 * k + 1, 5
        a = dev(2.0 + 0.1j * g.standard_normal(n))
        b = c = dev(np.full(n, -0.25 + 0.1j))
        if op == "mrhs":
            psi = normal(rhs, n)
            L = cn.Layout.contiguous(n, rhs, shared_coefficients=True)
            call = lambda p, out: cn.solve(a, b, c, p, out=out, layout=L)
        elif op == "solve":
            psi = normal(n)
            call = lambda p, out: cn.solve(a, b, c, p, out=out)
        else:
            x, psi = normal(n), normal(n)
            call = lambda p, out: cn.solve_adjoint(a, b, c, x, p, need_abc=False)[0]
    elif op == "uneven":
        lens = g.integers(1, 30000, 97)
        lens[0] = 40000 + k
        offs = np.concatenate([[0], np.cumsum(lens)]).astype(np.int64)
        L = cn.Layout.uneven(offs)
        psi, V = normal(int(offs[-1])), dev(g.uniform(-1.0, 0.0, int(offs[-1])))
        dxs = dev(g.uniform(0.1, 0.2, len(lens)))
        call = lambda p, out: cn.step(p, V, 0.0, 0.01, dx_per_system=dxs, out=out, layout=L)
    elif op == "absorbing":
        n = (1 << 18) + 37 * k + 1
        psi, V, W = normal(n), dev(g.uniform(-1.0, 0.0, n)), dev(g.uniform(0.0, 2.0, n))
        call = lambda p, out: cn.step(p, V, 0.1, 0.01, W=W, out=out)
    elif op == "rows":
        n, batch = 9001 + k, 40
        psi, V = normal(batch, n), dev(g.uniform(-1.0, 0.0, (batch, n)))
        call = lambda p, out: cn.step(p, V, 0.1, 0.01, out=out)
    else:
        n, batch = 1000 + k, 130
        psi, V = normal(n, batch), dev(g.uniform(-1.0, 0.0, (n, batch)))
        L = cn.Layout.interleaved(n, batch)
        dx = 0.1 if op == "columns" else 0.05  # kappa 0.25 (64-row tiles), 1.0 (128)
        call = lambda p, out: cn.step(p, V, dx, 0.01, out=out, layout=L)
    if nan:
        psi.view(-1)[psi.numel() // 2 + 11] = float("nan")
    want = call(psi, torch.empty_like(psi)).clone()
    torch.cuda.synchronize()
    cn.get_status()
    monkeypatch.setenv("CN_LINK_SPIN", str(spin))
    p = psi.clone()
    got = call(p, p if inplace else torch.empty_like(p))
    torch.cuda.synchronize()
    assert same(torch, got, want)
    assert cn.get_status() == (1 if nan else 0)
    monkeypatch.delenv("CN_LINK_SPIN")
    assert same(torch, call(psi, torch.empty_like(psi)), want)  # the next call
    cn.get_status()
