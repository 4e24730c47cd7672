"""Merge of shallow float32 volumes, which take one step of the one-A-scan kernel:
parity at both sides of the line, and the times of both sides."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every merge: float32 positions against float64 ones


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


@pytest.mark.parametrize("n,d", [(13, 61), (13, 62), (10, 60), (21, 5)])
def test_parity(octmc, n, d):
    log(f"merge of shallow float32 volumes n={n} d={d}")
    rng = np.random.default_rng(n + d)
    S, O = ([rng.uniform(0.1, 1.0, (n, n, d)).astype(np.float32) for _ in range(2)] for _ in range(2))
    V = [np.ones(n, np.float32) for _ in range(2)]
    D = rng.normal(0.0, 0.7, (2, n, n, 3)).astype(np.float32)
    D[0, 0, :2, 2] = (2000.0, -2000.0)
    D[1, 1, :3, 2] = (d, -d, -4.0)
    P = octmc.Pair(*(torch.from_numpy(x) for x in S), ox=torch.from_numpy(O[0]), oy=torch.from_numpy(O[1]),
                   vx=torch.from_numpy(V[0]), vy=torch.from_numpy(V[1]), dtype="f32", levels=1)
    mo, ma = (x.double().cpu().numpy() for x in P.merge(torch.from_numpy(D).cuda(), octa=True)[:2])
    P.close()
    ro, ra = oracle.merge(*(x.astype(np.float64) for x in (*S, D, *O, *V)))[:2]
    assert np.abs(mo - ro).max() < TOL * max(1.0, np.abs(ro).max())
    assert np.abs(ma - ra).max() < TOL * max(1.0, np.abs(ra).max())


def _best_us(run):
    for _ in range(20):
        run()
    best = float("inf")
    for _ in range(8):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        for _ in range(20):
            run()
        b.record()
        b.synchronize()
        best = min(best, a.elapsed_time(b) / 20 * 1e3)
    return best


@pytest.mark.parametrize("n", [200, 300])
def test_one_step_costs_less_than_two(octmc, n):
    """61 samples are one step of the one-A-scan kernel, 62 are one of the wider kernel's."""
    log(f"merge of float32 volumes of {n} x {n}: 61 and 62 samples")
    t = []
    for d in (61, 62):
        S = [torch.rand((n, n, d), device="cuda") for _ in range(2)]
        P = octmc.Pair(S[0], S[1], ox=S[0], oy=S[1], dtype="f32", levels=1)
        D = torch.randn((2, n, n, 3), device="cuda") * 0.3
        t.append(_best_us(lambda: P.merge(D, octa=True)))
        P.close()
    assert t[0] < 0.95 * t[1], t  # 0.99 by one kernel, 0.86 to 0.91 by the shorter loads
