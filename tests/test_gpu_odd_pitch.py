"""octmc_eval_noalloc of 16-bit volumes of many A-scans whose columns start at any
sample: odd depths (the caller's layout is not padded) and volumes that start an odd
number of samples into an allocation.  Against the oracle, at depths around the
windows of the matrix-core kernel, with fields whose windows start apart, and with a
last sample of the last A-scan that would be missed.  delta0 = 0 leaves the
angiographic term, which another kernel adds, out of the gradient."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import grad_err, log, rel, round_storage

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every evaluation: float32 kernels against the float64 oracle (tests/gpu_util.py)
T = {"bf16": torch.bfloat16, "f16": torch.float16}


@pytest.mark.parametrize("n,d,dtype,start,spread", [
    (91, 59, "bf16", 0, 0.6), (91, 59, "f16", 0, 9.0), (93, 123, "bf16", 0, 9.0), (91, 123, "f16", 0, 0.6),
    (91, 5, "bf16", 0, 3.0), (91, 117, "f16", 0, 3.0), (92, 58, "bf16", 1, 0.6), (91, 59, "f16", 1, 3.0),
    (92, 122, "bf16", 3, 9.0)])
def test_parity(n, d, dtype, start, spread):
    import paper_2010_06931_amd as octmc
    log(f"eval_noalloc n={n} d={d} {dtype} from sample {start}, displacements of {spread}")
    rng = np.random.default_rng(n + d + start)
    z = np.arange(d)
    edge = 0.4 * d + 2 * np.sin(np.arange(n) / 7.0)[:, None, None] + 2 * np.cos(np.arange(n) / 5.0)[None, :, None]
    S = []
    for _ in range(2):
        v = (0.1 + 0.8 / (1 + np.exp(-(z - edge) / 2.0))) * np.exp(0.4 * rng.normal(size=(n, n, d)))
        v[-1, -1, -1] = 40.0
        S.append(round_storage(torch.from_numpy(v.astype(np.float32)), dtype))
    A = [torch.from_numpy(rng.uniform(0, 1, (n, n)).astype(np.float32)) for _ in range(2)]
    V = [torch.ones(n) for _ in range(2)]
    V[0][n // 3] = V[1][n // 2] = 0.0
    D = torch.from_numpy((rng.uniform(-1, 1, (2, n, n, 3)) * spread).astype(np.float32))
    dev = []
    for s in S:
        buf = torch.zeros(start + s.numel(), dtype=T[dtype], device="cuda")
        buf[start:] = s.reshape(-1).cuda().to(T[dtype])
        dev.append(buf[start:].view(n, n, d))
    terms = torch.empty(octmc.NTERMS, dtype=torch.float64, device="cuda")
    eta = torch.zeros(1, dtype=torch.float64, device="cuda")
    grad = torch.empty((2, n, n, 3), device="cuda")
    octmc.eval_noalloc(*dev, *(x.cuda() for x in A + V), D.cuda(), eta, terms, grad, dtype=dtype,
                       params=octmc.default_params(delta0=0.0), eta_mode=0)
    t = octmc.terms_dict(terms)
    prm = oracle.Params(levels=1, delta0=0.0)
    lv = oracle.Level(*(x.double().numpy() for x in (*S, *A, *V)))
    D64 = D.double().numpy()
    ref_eta = oracle.eta_at(lv, D64, prm)
    ref, gref = oracle.evaluate(lv, D64, prm, ref_eta)
    g = grad.double().cpu().numpy()
    assert rel(t["eta"], ref_eta) < TOL
    for k in ("F", "data", "str", "str05"):
        assert rel(t[k], ref[k]) < TOL, (k, t[k], ref[k])
    assert grad_err(g, gref) < TOL
    assert grad_err(g[:, -1:, -1:], gref[:, -1:, -1:]) < TOL
