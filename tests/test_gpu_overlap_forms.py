"""The reverse mode of an interleaved batch run eagerly (the next segment recomputed on a second
stream) and replayed from a graph (segments one after the other) gives the same bits: both recompute
with the same form of the step.  kappa 0.25 and 1.0 step in one pass, 2.0 in two.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dx,dt", [(0.1, 0.01), (0.05, 0.01), (0.05, 0.02)])
def test_interleaved_adjoint(dx, dt):
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    n, batch, steps, K = 300, 130, 11, 3
    rng = np.random.default_rng(7)
    dev = lambda t: torch.from_numpy(t).cuda()
    tV, psi = dev(rng.uniform(-1, 0, (n, batch))), dev(workloads.complex_normal(rng, (n, batch)))
    gT = dev(workloads.complex_normal(rng, (n, batch)))
    L = cn.Layout.interleaved(n, batch)
    ckpt = torch.empty(-(-steps // K) * n * batch, dtype=torch.complex128, device="cuda")
    seg = torch.empty((K + 1) * n * batch, dtype=torch.complex128, device="cuda")
    cn.propagate(psi, tV, dx, dt, steps, ckpt=ckpt, K=K, layout=L)

    def run(g, dV):
        cn.propagate_adjoint(ckpt, g, tV, dx, dt, steps, K, dV=dV, seg=seg, layout=L)

    ge, dVe = gT.clone(), torch.zeros_like(tV)
    run(ge, dVe)
    torch.cuda.synchronize()
    gc, dVc = gT.clone(), torch.zeros_like(tV)
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=side):
        run(gc, dVc)
    for _ in range(3):
        gc.copy_(gT)
        dVc.zero_()
        graph.replay()
        torch.cuda.synchronize()
        run(gT.clone(), torch.zeros_like(tV))  # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(gc, ge) and torch.equal(dVc, dVe)
    assert cn.get_status() == 0
