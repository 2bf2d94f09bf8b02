"""One-pass steps of an interleaved batch whose off-diagonal changes from call to call on one layout
(a time-step study, half and full steps of a splitting, grids of two spacings): kappa 0.25 takes
tiles of 64 rows, 1.0 tiles of 128, and each tile size keeps line buffers of its own.  Every call is
compared with the CPU oracle: relative L2 <= 1e-11 per system, as everywhere.
"""
import numpy as np
import pytest

import workloads

pytestmark = pytest.mark.gpu
TOL = 1e-11
GRID = {0.25: (0.1, 0.01), 1.0: (0.05, 0.01)}  # kappa: (dx, dt)


@pytest.fixture(scope="module")
def gpu():
    torch = pytest.importorskip("torch")
    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    import paper_2205_00856_amd as cn

    cn.handle(0)
    return torch, cn


@pytest.fixture(scope="module")
def data(oracle_mod):
    """Per layout: V, psi and the oracle's step for either kappa."""
    made = {}

    def get(n, batch):
        if (n, batch) not in made:
            g = np.random.default_rng(n + batch)
            V, psi = g.uniform(-2.0, 2.0, (n, batch)), workloads.complex_normal(g, (n, batch))
            ref = {k: np.stack([oracle_mod.cn_step(psi[:, s], V[:, s], *GRID[k])
                                for s in range(batch)], 1) for k in GRID}
            made[n, batch] = V, psi, ref
        return made[n, batch]

    return get


def close(got, ref):
    err = np.linalg.norm(got.cpu().numpy() - ref, axis=0)
    assert (err <= TOL * np.linalg.norm(ref, axis=0)).all(), err.max()


# each run of calls: every switch from either tile size after odd and even counts of passes
@pytest.mark.parametrize("runs", [(1, 1, 1, 1), (2, 2, 1, 2), (1, 2, 3, 1), (3, 3, 2, 1)])
@pytest.mark.parametrize("n,batch", [(129, 64), (1009, 200), (2500, 130)])
@pytest.mark.parametrize("first", [0.25, 1.0])
def test_switch(gpu, data, first, n, batch, runs):
    torch, cn = gpu
    V, psi, ref = data(n, batch)
    tV, p0 = torch.from_numpy(V).cuda(), torch.from_numpy(psi).cuda()
    L = cn.Layout.interleaved(n, batch)
    kaps = [first, 1.25 - first] * 2
    outs = []
    for kap, count in zip(kaps, runs):
        dx, dt = GRID[kap]
        for _ in range(count):
            p = p0.clone()
            cn.step(p, tV, dx, dt, out=p, layout=L)
            outs.append((kap, p))
    for kap, p in outs:
        close(p, ref[kap])
    assert cn.get_status() == 0


@pytest.mark.parametrize("graph", [0.25, 1.0])
def test_switch_around_replays(gpu, data, graph):
    torch, cn = gpu
    n, batch = 1009, 200
    V, psi, ref = data(n, batch)
    tV, p0 = torch.from_numpy(V).cuda(), torch.from_numpy(psi).cuda()
    L = cn.Layout.interleaved(n, batch)
    eager = 1.25 - graph
    cn.step(p0, tV, *GRID[eager], layout=L)
    out = torch.empty_like(p0)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        cn.step(p0, tV, *GRID[graph], out=out, layout=L)
    for count in (1, 2, 1, 3):
        out.fill_(7.0)
        g.replay()
        torch.cuda.synchronize()
        close(out, ref[graph])
        for _ in range(count):
            close(cn.step(p0, tV, *GRID[eager], layout=L), ref[eager])
    assert cn.get_status() == 0
