"""The matrix-core structural kernels (16-bit volumes of at least 8192 A-scans; a
pair, and three or four volumes) and merge (volumes of at least 8192 A-scans)
against the FP64 oracle, at the sizes and fields where its tiling can go wrong:
scans that are no multiple of its 4 x 4 blocks and 2 x 2 tiles, depths around
its windows of 16 x 4 and 16 x 8 samples (58 and 122 outputs a step, the
smallest depths), tiles whose A-scans share all, some or none of their source
columns, depth offsets that differ within a tile, and samples that are not
finite.  delta0 = 0 leaves the angiographic term, which another kernel adds,
out of the gradient."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import grad_err, log, rel, round_storage

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every evaluation: float32 kernels against the float64 oracle (tests/gpu_util.py)


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


def _inputs(n, d, dtype, seed, count=2):
    """Speckled layers, en face images and validity with one invalid B-scan each."""
    rng = np.random.default_rng(seed)
    z = np.arange(d)[None, None, :]
    edge = 0.4 * d + 2 * np.sin(np.arange(n) / 7.0)[:, None, None] + 2 * np.cos(np.arange(n) / 5.0)[None, :, None]
    vol = [(0.1 + 0.8 / (1 + np.exp(-(z - edge) / 2.0))) * np.exp(0.4 * rng.normal(size=(n, n, d))) for _ in range(count)]
    S = [round_storage(torch.from_numpy(v.astype(np.float32)), dtype) for v in vol]
    A = [torch.from_numpy(rng.uniform(0, 1, (n, n)).astype(np.float32)) for _ in range(count)]
    V = [torch.ones(n) for _ in range(count)]
    for q in range(count):
        V[q][n // (3 - q % 2)] = 0.0
    return S, A, V


def _field(case, n, seed, count=2):
    rng = np.random.default_rng(seed + 100)
    D = np.zeros((count, n, n, 3))
    if case == "shift":      # whole samples: every fraction 0, odd and even depth offsets
        D[0] += (1.0, -2.0, 3.0)
        D[1] += (-1.0, 0.0, -2.0)
    elif case == "noise":    # neighbours differ by about a pixel
        D += rng.normal(0.0, 0.6, D.shape)
    elif case == "depth":    # depth offsets of a tile up to eight samples apart, and beyond both ends
        D[..., 2] = rng.uniform(-8.0, 8.0, D.shape[:3])
        D[..., 2][rng.uniform(size=D.shape[:3]) < 0.01] = 2000.0
        D[..., 2][rng.uniform(size=D.shape[:3]) < 0.01] = -2000.0
    elif case == "apart":    # disjoint stencils: more columns than one pass holds; some outside the scan
        D += rng.uniform(-9.0, 9.0, D.shape)
    return torch.from_numpy(D.astype(np.float32))


def _eval(octmc, n, d, dtype, S, A, V, D):
    P = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype=dtype, levels=1, delta0=0.0)
    terms, g = P.eval(0, D.cuda(), eta_mode=0)
    t = octmc.terms_dict(terms)
    g = g.double().cpu().numpy()
    P.close()
    return t, g


@pytest.mark.parametrize("n,d,dtype,case", [
    (91, 122, "bf16", "noise"), (92, 123, "f16", "noise"), (93, 244, "bf16", "apart"), (94, 245, "f16", "depth"),
    (91, 58, "bf16", "apart"), (93, 59, "f16", "noise"), (91, 117, "bf16", "depth"), (92, 233, "bf16", "shift"),
    (91, 4, "bf16", "noise"), (91, 7, "f16", "depth"), (91, 8, "bf16", "apart"), (95, 465, "bf16", "noise"),
    (200, 4, "f32", "noise"), (201, 58, "f32", "apart"), (203, 62, "f32", "depth"), (200, 116, "f32", "shift"),
    (201, 174, "f32", "noise"),
])
def test_parity(octmc, n, d, dtype, case):
    log(f"matrix-core structural kernel n={n} d={d} {dtype} {case}")
    S, A, V = _inputs(n, d, dtype, n + d)
    D = _field(case, n, n + d)
    t, g = _eval(octmc, n, d, dtype, S, A, V, D)
    prm = oracle.Params(levels=1, delta0=0.0)
    lv = oracle.Level(*(x.double().numpy() for x in (S[0], S[1], A[0], A[1], V[0], V[1])))
    D64 = D.double().numpy()
    eta = oracle.eta_at(lv, D64, prm)
    ref, gref = oracle.evaluate(lv, D64, prm, eta)
    assert rel(t["eta"], eta) < TOL
    for k in ("F", "data", "str", "str05"):
        assert rel(t[k], ref[k]) < TOL, (k, t[k], ref[k])
    assert grad_err(g, gref) < TOL


@pytest.mark.parametrize("value", [float("nan"), float("inf")])
def test_not_finite_stays_local(octmc, value):
    """A sample that is not finite reaches the A-scans whose stencil holds its
    column and no others of their tile."""
    n, d = 91, 130
    log(f"matrix-core structural kernel with a sample of {value}")
    S, A, V = _inputs(n, d, "bf16", 5)
    D = _field("noise", n, 5)
    r, c = 40, 33
    S[0][r, c, 60] = value
    P = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype="bf16", levels=1)
    _, g = P.eval(0, D.cuda(), eta_mode=1)  # the stored eta: one from these volumes would not be finite
    g = g.double().cpu().numpy()
    P.close()
    f = np.floor(D[0].double().numpy()).astype(int)
    jj, ii = np.mgrid[0:n, 0:n]
    hit = np.zeros((n, n), bool)
    for b in range(4):
        for a in range(4):
            hit |= (np.clip(jj + f[..., 1] - 1 + b, 0, n - 1) == r) & (np.clip(ii + f[..., 0] - 1 + a, 0, n - 1) == c)
    bad = ~np.isfinite(g).all(axis=(0, 3))
    assert hit.sum() > 4 and (bad == hit).all()


@pytest.mark.parametrize("n,d,dtype,count,case", [
    (91, 58, "bf16", 3, "noise"), (92, 59, "f16", 4, "depth"), (93, 117, "bf16", 4, "apart"), (91, 4, "f16", 3, "depth"),
    (94, 130, "bf16", 4, "noise"), (200, 58, "f32", 4, "noise"), (201, 62, "f32", 4, "apart"), (203, 4, "f32", 4, "depth"),
])
def test_parity_multi(octmc, n, d, dtype, count, case):
    log(f"matrix-core structural kernel of {count} volumes n={n} d={d} {dtype} {case}")
    S, A, V = _inputs(n, d, dtype, n + d, count)
    D = _field(case, n, n + d, count)
    orient = [0, 1, 0, 1][:count]
    M = octmc.Multi(S, orient, enface=A, valid=V, dtype=dtype, levels=1, delta0=0.0)
    terms, g = M.eval(0, D.cuda(), eta_mode=0)
    t = octmc.terms_dict(terms)
    g = g.double().cpu().numpy()
    M.close()
    prm = oracle.Params(levels=1, delta0=0.0)
    om = oracle.Multi([s.double().numpy() for s in S], orient, [a.double().numpy() for a in A],
                      [v.double().numpy() for v in V])
    D64 = D.double().numpy()
    _, p05, _ = oracle.evaluate_multi(om, D64, prm, None, grad=False)
    eta = np.sqrt(p05[:, 1] / p05[:, 0])
    ref, _, gref = oracle.evaluate_multi(om, D64, prm, eta)
    for k in ("F", "data", "str", "str05"):
        assert rel(t[k], ref[k]) < TOL, (k, t[k], ref[k])
    assert grad_err(g, gref) < TOL


@pytest.mark.parametrize("n,d,dtype,case", [
    (91, 122, "bf16", "noise"), (92, 123, "f16", "apart"), (93, 60, "f32", "noise"), (94, 121, "f32", "apart"),
    (91, 59, "bf16", "depth"), (91, 4, "f32", "depth"), (92, 7, "f16", "noise"), (93, 233, "f32", "shift"),
])
def test_parity_merge(octmc, n, d, dtype, case):
    log(f"matrix-core merge n={n} d={d} {dtype} {case}")
    S, A, V = _inputs(n, d, dtype, n + d)
    O, _, _ = _inputs(n, d, "f32", n + d + 1)
    D = _field(case, n, n + d)
    P = octmc.Pair(S[0], S[1], ox=O[0], oy=O[1], vx=V[0], vy=V[1], dtype=dtype, levels=1)
    mo, ma = P.merge(D.cuda(), octa=True)
    mo, ma = mo.double().cpu().numpy(), ma.double().cpu().numpy()
    P.close()
    Os = [oracle.substitute_invalid(O[q], V[q], q) for q in range(2)]
    ro, ra, _, _ = oracle.merge(S[0].double(), S[1].double(), D.double(), Os[0], Os[1], V[0].double(), V[1].double(),
                                P.params.merge_kappa, P.params.merge_tau)
    # float32 positions of order 100 put the densities, and with them the
    # weights, some 1e-5 off; the bar of every merge
    assert np.abs(mo - ro).max() < TOL * max(1.0, np.abs(ro).max())
    assert np.abs(ma - ra).max() < TOL * max(1.0, np.abs(ra).max())


def test_merge_not_finite_stays_local(octmc):
    n, d = 91, 130
    log("matrix-core merge with a sample that is not a number")
    S, A, V = _inputs(n, d, "bf16", 5)
    D = _field("noise", n, 5)
    r, c = 40, 33
    S[0][r, c, 60] = float("nan")
    P = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype="bf16", levels=1)
    mo, _ = P.merge(D.cuda())
    mo = mo.cpu().numpy()
    P.close()
    f = np.floor(D[0].double().numpy()).astype(int)
    jj, ii = np.mgrid[0:n, 0:n]
    hit = np.zeros((n, n), bool)
    for b in range(4):
        for a in range(4):
            hit |= (np.clip(jj + f[..., 1] - 1 + b, 0, n - 1) == r) & (np.clip(ii + f[..., 0] - 1 + a, 0, n - 1) == c)
    bad = np.isnan(mo)
    assert hit.sum() > 4 and (bad.any(axis=2) == hit).all() and (bad[hit].sum(axis=1) == 4).all()
