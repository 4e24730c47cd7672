"""Merge of 16-bit volumes of many A-scans with a sample that is infinite: the
outputs whose stencils hold it are infinite, with the sign of its weight, and no
others change.  (Binary16 storage makes an infinity of every value beyond 65504.)"""
import numpy as np
import pytest
import torch

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


def _taps(t):
    """Catmull-Rom weights of the samples n - 1 .. n + 2."""
    return np.stack([-t * (1 - t) ** 2, 2 - 5 * t ** 2 + 3 * t ** 3, t + 4 * t ** 2 - 3 * t ** 3, -t ** 2 * (1 - t)]) / 2


def _weight(D, n, d, at):
    """[n][n][d]: the weight of the sample at = (row, column, depth) in every output of one scan."""
    f = np.floor(D)
    t = _taps(D - f)  # [4][n][n][3]
    jj, ii = np.mgrid[0:n, 0:n]
    W = np.ones((n, n, d))
    for axis, pos in ((0, ii), (1, jj)):
        e = at[1 - axis] - (pos + f[..., axis].astype(int) - 1)
        v = np.take_along_axis(t[..., axis], np.clip(e, 0, 3)[None], 0)[0]
        W *= np.where((e >= 0) & (e < 4), v, 0.0)[..., None]
    e = at[2] - (np.arange(d)[None, None] + f[..., 2:3].astype(int) - 1)
    v = np.choose(np.clip(e, 0, 3), [t[q][..., 2:3] for q in range(4)])
    return W * np.where((e >= 0) & (e < 4), v, 0.0)


@pytest.mark.parametrize("dtype,value,spread", [("f16", 70000.0, 0.6), ("f16", float("-inf"), 9.0),
                                                ("bf16", float("inf"), 9.0), ("bf16", float("-inf"), 0.6)])
def test_infinite_sample(octmc, dtype, value, spread):
    n, d, at = 91, 130, (40, 33, 60)
    log(f"merge of {dtype} volumes with a sample of {value}, displacements of {spread}")
    g = torch.Generator().manual_seed(11)
    S = [torch.rand((n, n, d), generator=g) + 0.1 for _ in range(2)]
    A = torch.rand((n, n), generator=g)
    D = torch.randn((2, n, n, 3), generator=g).clamp(-3, 3) * spread
    out = []
    for v in (0.5, value):
        S[1][at] = v
        P = octmc.Pair(S[0], S[1], ax=A, ay=A, dtype=dtype, levels=1, merge_tau=0.0)
        mo, _ = P.merge(D.cuda())
        out.append(mo.cpu().numpy())
        P.close()
    W = _weight(D[1].double().numpy(), n, d, at)
    hit = W != 0
    assert hit.sum() > 16
    # the merge weights are positive (merge_tau = 0: none is cut off)
    assert (out[1][hit] == np.sign(W[hit]) * np.copysign(np.inf, value)).all()
    assert np.isfinite(out[1][~hit]).all()
    # a float32 sum of 128 products against the same in another order
    assert np.abs(out[1][~hit] - out[0][~hit]).max() < 128 * 2.0 ** -24 * np.abs(out[0]).max() * 4
