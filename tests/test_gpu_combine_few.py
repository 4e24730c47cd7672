"""The combination kernel of few A-scans (at most 8192) against the FP64 oracle:
scans whose A-scans do not fill its last block of 32 or its displacement sums of
four, one block and all of them, both sides of the line to the kernel of many
A-scans; and the count that finds its last block, over repeats, passes that write
eta first, evaluations of other sizes in the same scratch, and graph replays."""
import numpy as np
import pytest
import torch

import oracle
from gpu_util import grad_err, log, rel

pytestmark = pytest.mark.gpu

TOL = 1e-4  # the bar of every evaluation: float32 kernels against the float64 oracle (tests/gpu_util.py)


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


def _inputs(n, d, seed):
    rng = np.random.default_rng(seed)
    S = [torch.from_numpy(rng.uniform(0.1, 1.0, (n, n, d)).astype(np.float32)) for _ in range(2)]
    x = np.arange(n) / 9.0
    base = 0.3 * np.sin(x)[:, None] * np.cos(1.3 * x)[None, :]
    # en face images well apart: their difference stays clear of the loss's kink
    A = [torch.from_numpy((base + 0.6 * q).astype(np.float32)) for q in range(2)]
    V = [torch.ones(n), torch.ones(n)]
    V[0][n // 2] = V[1][n // 3] = 0.0
    D = torch.from_numpy(rng.normal(0.0, 0.8, (2, n, n, 3)).astype(np.float32))
    return S, A, V, D


@pytest.mark.parametrize("n,d", [(4, 8), (5, 8), (7, 9), (11, 16), (33, 12), (64, 8), (89, 5), (90, 8), (91, 8)])
def test_parity(octmc, n, d):
    log(f"combination of few A-scans n={n} d={d}")
    S, A, V, D = _inputs(n, d, n)
    P = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], vx=V[0], vy=V[1], dtype="f32", levels=1)
    prm = oracle.Params(levels=1)
    lv = oracle.Level(*(x.double().numpy() for x in (S[0], S[1], A[0], A[1], V[0], V[1])))
    D64 = D.double().numpy()
    eta = oracle.eta_at(lv, D64, prm)
    ref, gref = oracle.evaluate(lv, D64, prm, eta)
    first = None
    for mode in (0, 1, 1, 0):  # the stored eta is this displacement's after the first
        terms, g = P.eval(0, D.cuda(), eta_mode=mode)
        t = octmc.terms_dict(terms)
        assert rel(t["eta"], eta) < TOL
        for k in ("F", "data", "str", "ang", "reg", "mean", "str05", "ang05"):
            assert rel(t[k], ref[k]) < TOL, (k, t[k], ref[k])
        assert grad_err(g.double().cpu().numpy(), gref) < TOL
        first = (terms.clone(), g.clone()) if first is None else first
        assert torch.equal(terms, first[0]) and torch.equal(g, first[1])
    P.close()


def test_sizes_in_turn_in_one_scratch_and_replayed(octmc):
    """Evaluations of few and of many A-scans one after the other in the static
    scratch, then the same captured and replayed."""
    sets = []
    for n, d in ((24, 16), (90, 8), (120, 8), (9, 12)):
        S, A, V, D = _inputs(n, d, n)
        ins = [x.cuda() for x in (*S, *A, *V)]
        eta, terms = torch.ones(1, dtype=torch.float64, device="cuda"), torch.zeros(octmc.NTERMS, dtype=torch.float64, device="cuda")
        grad = torch.zeros((2, n, n, 3), device="cuda")
        sets.append((ins, D.cuda(), eta, terms, grad))

    def all_of_them():
        for ins, D, eta, terms, grad in sets:
            octmc.eval_noalloc(*ins, D, eta, terms, grad, eta_mode=0)

    octmc.context()
    log("few and many A-scans in turn, eager")
    all_of_them()
    torch.cuda.synchronize()
    want = [(t.clone(), g.clone()) for _, _, _, t, g in sets]
    for k, (ins, D, _, terms, grad) in enumerate(sets):
        P = octmc.Pair(ins[0], ins[1], ax=ins[2], ay=ins[3], vx=ins[4], vy=ins[5], dtype="f32", levels=1)
        t, g = P.eval(0, D, eta_mode=0)
        assert torch.equal(t, want[k][0]) and torch.equal(g, want[k][1])
        P.close()
    stream = torch.cuda.Stream()
    stream.wait_stream(torch.cuda.current_stream())
    graph = torch.cuda.CUDAGraph()
    log("few and many A-scans in turn, captured")
    with torch.cuda.graph(graph, stream=stream):
        all_of_them()
    for _ in range(4):
        for _, _, _, terms, grad in sets:
            terms.zero_()
            grad.zero_()
        graph.replay()
        torch.cuda.synchronize()
        for (_, _, _, terms, grad), (t, g) in zip(sets, want):
            assert torch.equal(terms, t) and torch.equal(grad, g)
        all_of_them()
        torch.cuda.synchronize()
