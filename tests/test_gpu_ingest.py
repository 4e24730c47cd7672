"""Ingest against the FP64 oracle at the sizes where its kernels' loads and stores
end: odd and even scans, depths of every remainder of four and beyond the rows' 512
samples, padded storage, replaced B-scans (the first, the last, neighbours, all but
one), from device and from host memory."""
import ctypes as C

import numpy as np
import pytest
import torch

import oracle
from gpu_util import grad_err, log, rel

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every evaluation: float32 kernels against the float64 oracle (tests/gpu_util.py)


def _scans(n, d, seed):
    rng = np.random.default_rng(seed)
    S = [rng.uniform(0.1, 1.0, (n, n, d)).astype(np.float32) for _ in range(2)]
    # OCTA volumes well apart, so that the en face loss stays clear of its kink
    O = [(rng.uniform(0.1, 1.0, (n, n, d)) + 2.0 * q).astype(np.float32) for q in range(2)]
    V = [np.ones(n, np.float32), np.ones(n, np.float32)]
    V[0][[0, 1, n - 1]] = 0.0
    V[1][:] = 0.0
    V[1][n // 2] = 1.0
    return S, O, V


@pytest.mark.parametrize("n,d,dtype", [(7, 8, "f32"), (8, 9, "f32"), (9, 10, "bf16"), (10, 11, "bf16"), (7, 7, "bf16"),
                                       (16, 64, "f32"), (9, 513, "f32"), (8, 527, "bf16")])
def test_levels_and_octa(n, d, dtype):
    import paper_2010_06931_amd as octmc
    log(f"ingest n={n} d={d} {dtype}")
    S, O, V = _scans(n, d, n + d)
    sub = [oracle.substitute_invalid(O[q].astype(np.float64), V[q].astype(np.float64), q) for q in range(2)]
    img = [oracle.enface_mean(x) for x in sub]
    lv = oracle.level_from(*(x.astype(np.float64) for x in S), *img, *(v.astype(np.float64) for v in V))
    pyr = oracle.pyramid(lv, 2, store=0 if dtype == "f32" else 1)
    P = octmc.Pair(*(torch.from_numpy(x) for x in S), ox=torch.from_numpy(O[0]), oy=torch.from_numpy(O[1]),
                   vx=torch.from_numpy(V[0]), vy=torch.from_numpy(V[1]), dtype=dtype, levels=2)
    prm = oracle.Params(levels=2)
    for level in (0, 1):
        m = n if level == 0 else (n + 1) // 2
        D = np.random.default_rng(m).normal(0.0, 0.5, (2, m, m, 3)).astype(np.float32)
        terms, g = P.eval(level, torch.from_numpy(D).cuda(), eta_mode=0)
        t = octmc.terms_dict(terms)
        D64 = D.astype(np.float64)
        eta = oracle.eta_at(pyr[level], D64, prm)
        ref, gref = oracle.evaluate(pyr[level], D64, prm, eta)
        assert rel(t["eta"], eta) < TOL
        for k in ("F", "data", "str", "ang"):
            assert rel(t[k], ref[k]) < TOL, (level, k, t[k], ref[k])
        assert grad_err(g.double().cpu().numpy(), gref) < TOL
    # the volumes kept for the merge: at rest each merged OCTA sample is a blend of them
    Z = torch.zeros((2, n, n, 3), device="cuda")
    merged = P.merge(Z, octa=True)[1].double().cpu().numpy()
    P.close()
    want = oracle.merge(*(x.astype(np.float64) for x in S), np.zeros((2, n, n, 3)), *sub,
                        *(v.astype(np.float64) for v in V))[1]
    assert np.abs(merged - want).max() <= TOL * np.abs(want).max()


def test_host_inputs_give_the_same_bits():
    import paper_2010_06931_amd as octmc
    n, d = 13, 21
    S, O, V = _scans(n, d, 3)
    P = octmc.Pair(*(torch.from_numpy(x).cuda() for x in S), ox=torch.from_numpy(O[0]).cuda(), oy=torch.from_numpy(O[1]).cuda(),
                   vx=torch.from_numpy(V[0]).cuda(), vy=torch.from_numpy(V[1]).cuda(), dtype="f32", levels=2)
    L = octmc.lib()
    shape = octmc.Shape(n, n, d, octmc.F32, octmc.MEM_HOST)
    prm = octmc.default_params()
    prm.levels = 2
    vp = lambda x: x.ctypes.data_as(C.c_void_p)
    h = C.c_void_p()
    log("ingest from host memory")
    rc = L.octmc_pair_create(octmc.context()._h, C.byref(prm), C.byref(shape), vp(S[0]), vp(S[1]), vp(O[0]), vp(O[1]),
                             None, None, vp(V[0]), vp(V[1]), None, C.byref(h))
    assert rc == 0
    want = P.merge(torch.zeros((2, n, n, 3), device="cuda"), octa=True)
    D = torch.from_numpy(np.random.default_rng(1).normal(0.0, 0.5, (2, n, n, 3)).astype(np.float32)).cuda()
    tw, gw = P.eval(0, D, eta_mode=0)
    device, P._h = P._h, h
    got = P.merge(torch.zeros((2, n, n, 3), device="cuda"), octa=True)
    tg, gg = P.eval(0, D, eta_mode=0)
    P.close()
    P._h = device
    P.close()
    for a, b in ((want[0], got[0]), (want[1], got[1]), (tw, tg), (gw, gg)):
        assert torch.equal(a, b)
