"""The walks of the en face filters against the FP64 oracle, voxel counts exactly,
at the lengths where a walk ends or begins: positions around its chunks of 15 and
its segments, depths around its tiles of 62 and 64 samples, one and two lines,
and so few samples that the order statistics have prefixes of their own."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import log

pytestmark = pytest.mark.gpu

TOL = 1e-6  # float32 results of float64 means and medians of exactly selected samples


@pytest.mark.parametrize("shape", [(2, 7, 61), (3, 8, 62), (9, 15, 63), (8, 16, 64), (16, 30, 124), (17, 31, 125),
                                   (45, 46, 2), (61, 60, 1), (3100, 105, 2), (1600, 215, 1), (106, 3100, 3),
                                   (1, 1, 21), (1, 2, 40)])
def test_filters_at_the_ends_of_their_walks(shape):
    import paper_2010_06931_amd as octmc
    h, w, d = shape
    rng = np.random.default_rng(h + 10 * w + 100 * d)
    s = rng.random(shape, dtype=np.float32)
    a = rng.normal(size=shape).astype(np.float32)
    for V in (0, 1):
        log(f"en face walk {shape} scan {V}")
        out, cnt, st = octmc.enface_project(torch.from_numpy(s).cuda(), torch.from_numpy(a).cuda(), V, details=True)
        ref, rcnt, rst = oracle.enface_project(s, a, V, None, details=True)
        assert np.array_equal(cnt.cpu().numpy(), rcnt.astype(np.int32))
        assert st[0] == rst[0] and st[1] == rst[1] and st[2] == rst[2]
        assert (np.abs(out.cpu().numpy() - ref) / (1 + np.abs(ref))).max() <= TOL
