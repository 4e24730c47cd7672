"""Axial resampling against the FP64 oracle at the depths where its loads and stores
of four samples end, with shifts inside, at and beyond both ends of the A-scan."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log

pytestmark = pytest.mark.gpu

# float32: the weights are cubics of an exact fraction (three roundings of terms up
# to 3), four products of them with samples up to 1 are added
TOL = 4e-6


@pytest.mark.parametrize("h,w,d", [(3, 5, 1), (3, 5, 2), (4, 4, 3), (7, 5, 4), (6, 5, 7), (9, 8, 8), (9, 8, 9), (5, 4, 63),
                                   (5, 4, 64), (5, 7, 65), (4, 5, 257), (3, 4, 516)])
def test_ends_of_the_rows(h, w, d):
    import paper_2010_06931_amd as octmc
    rng = np.random.default_rng(d)
    vol = rng.random((h, w, d), dtype=np.float32)
    dz = rng.uniform(-(d + 3.0), d + 3.0, (h, w)).astype(np.float32)
    dz[0, :4] = (0.0, 0.5, -0.25, -1.0)
    dz[1, :4] = (d, -d, 1e9, -1e9)
    dz[2, :3] = (d - 4.0, 3.75, -3.25)
    log(f"axial resampling {h}x{w}x{d}")
    got = octmc.resample_axial(torch.from_numpy(vol).cuda(), torch.from_numpy(dz).cuda()).cpu().numpy()
    want = oracle.resample_z(vol.astype(np.float64), dz.astype(np.float64))
    assert np.abs(got - want).max() <= TOL
