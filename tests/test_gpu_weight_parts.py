"""The smallest lateral weights of the matrix-core kernels with binary16 storage: a
merged value that is one small weight times one sample."""
import numpy as np
import pytest
import torch

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_small_weight(dtype):
    import paper_2010_06931_amd as octmc
    n, d, gap = 96, 24, 6
    log(f"merge of {dtype} volumes by weights below 2^-13")
    rng = np.random.default_rng(3)
    t = (2.0 ** rng.uniform(-8.5, -6.0, (n, n, 2))).astype(np.float32)
    D = np.zeros((2, n, n, 3), np.float32)
    D[..., :2] = t
    S = torch.zeros((n, n, d))
    S[::gap, ::gap] = 1.0
    # the A-scans one row and one column on: their first taps alone meet a column that is not 0
    P = octmc.Pair(S, S, ax=torch.ones((n, n)), ay=torch.ones((n, n)), dtype=dtype, levels=1)
    mo = P.merge(torch.from_numpy(D).cuda())[0].double().cpu().numpy()[1::gap, 1::gap]
    P.close()
    t = t.astype(np.float64)[1::gap, 1::gap]
    w = np.prod(-t * (1 - t) ** 2 / 2, axis=-1)[..., None]
    assert w.min() < 2.0 ** -18 and w.max() < 2.0 ** -13
    # the split's bound, and 2^-21 for the roundings of the taps, products and sums (some eight of 2^-24)
    assert (np.abs(mo - w) <= 2.0 ** -40 + w * 2.0 ** -21).all(), np.abs(mo / w - 1).max()
