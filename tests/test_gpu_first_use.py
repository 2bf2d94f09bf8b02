"""The first call on a layout, on a non-blocking stream while the default stream is busy: the memory
that the new plan sets up (line buffers, marks) is ready before the first pass runs, whatever the
stream.  Against the CPU oracle: relative L2 <= 1e-11.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-11


def rel(got, ref):
    return float(np.linalg.norm(got.cpu().numpy() - ref) / np.linalg.norm(ref))


@pytest.mark.parametrize("op", ["solve", "rows", "columns"])
def test_first_call_beside_a_busy_default_stream(oracle_mod, op):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    g = np.random.default_rng(5)
    if op == "solve":  # 1024 tiles of 512 rows
        n, batch = (1 << 19) + 1234, 1
        a = 2.0 + 0.1j * g.standard_normal(n)
        b = c = np.full(n, -0.25 + 0.1j)
        d = workloads.complex_normal(g, n)
        ref = oracle_mod.thomas(a, b, c, d)
        args = [torch.from_numpy(t).cuda() for t in (a, b, c, d)]
    else:  # 5 tiles of 2048 rows a system; 20 tiles of 64 rows
        n, batch = (9001, 40) if op == "rows" else (1234, 140)
        V, psi = g.uniform(-2.0, 0.0, (batch, n)), workloads.complex_normal(g, (batch, n))
        ref = np.stack([oracle_mod.cn_step(psi[s], V[s], 0.1, 0.01) for s in range(batch)])
        if op == "columns":
            V, psi, ref = V.T.copy(), psi.T.copy(), ref.T
        args = [torch.from_numpy(t).cuda() for t in (psi, V)]
    side = torch.cuda.Stream()
    work = torch.ones(6000, 6000, dtype=torch.float64, device="cuda")
    out = torch.empty_like(args[-1] if op == "solve" else args[0])
    torch.cuda.synchronize()
    for _ in range(8):  # some 50 ms on the default stream
        work = work @ work * 1e-4
    with torch.cuda.stream(side):
        if op == "solve":
            cn.solve(*args, out=out)
        else:
            L = cn.Layout.contiguous(n, batch) if op == "rows" else cn.Layout.interleaved(n, batch)
            cn.step(*args, 0.1, 0.01, out=out, layout=L)
    side.synchronize()
    assert rel(out, ref) <= TOL
    torch.cuda.synchronize()
