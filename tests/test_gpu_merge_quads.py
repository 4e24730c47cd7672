"""The merge of float32 volumes against the FP64 oracle where its steps of 252 outputs
and its loads of four samples end, on scans that are no multiple of its 2 x 2 tiles,
with depth offsets inside, across and far beyond both ends of the A-scans."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every merge: float32 positions against float64 ones


@pytest.mark.parametrize("n,d", [(4, 4), (5, 7), (9, 251), (6, 252), (7, 253), (5, 504), (8, 505), (33, 33)])
def test_parity(n, d):
    import paper_2010_06931_amd as octmc
    log(f"merge of float32 volumes n={n} d={d}")
    rng = np.random.default_rng(n + d)
    S, O = ([rng.uniform(0.1, 1.0, (n, n, d)).astype(np.float32) for _ in range(2)] for _ in range(2))
    V = [np.ones(n, np.float32) for _ in range(2)]
    D = rng.normal(0.0, 0.7, (2, n, n, 3)).astype(np.float32)
    D[..., 2] = rng.uniform(-9.0, 9.0, (2, n, n))
    D[0, 0, :2, 2] = (2000.0, -2000.0)
    D[1, 1, :3, 2] = (d, -d, -4.0)
    P = octmc.Pair(*(torch.from_numpy(x) for x in S), ox=torch.from_numpy(O[0]), oy=torch.from_numpy(O[1]),
                   vx=torch.from_numpy(V[0]), vy=torch.from_numpy(V[1]), dtype="f32", levels=1)
    mo, ma = (x.double().cpu().numpy() for x in P.merge(torch.from_numpy(D).cuda(), octa=True)[:2])
    P.close()
    ro, ra = oracle.merge(*(x.astype(np.float64) for x in (*S, D, *O, *V)))[:2]
    assert np.abs(mo - ro).max() < TOL * max(1.0, np.abs(ro).max())
    assert np.abs(ma - ra).max() < TOL * max(1.0, np.abs(ra).max())
