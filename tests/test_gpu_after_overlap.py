"""Evaluations of few A-scans that overlap on one object (a mistake of the caller's:
they share its scratch) spoil their own results at most: every later evaluation
has the bits of one that nothing overlapped.  The count of finished blocks, by
which the last block of a combination forms the sums, is the state at stake."""
import pytest
import torch

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


def _overlap(runs):
    """Every run many times, each on a stream of its own, without an order between them."""
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in runs]
    for _ in range(40):
        for run, s in zip(runs, streams):
            with torch.cuda.stream(s):
                run()
    torch.cuda.synchronize()


def _scans(n, d, count=2):
    g = torch.Generator().manual_seed(n + d)
    S = [torch.rand((n, n, d), generator=g).cuda() for _ in range(count)]
    A = [torch.rand((n, n), generator=g).cuda() for _ in range(count)]
    return S, A, (torch.randn((count, n, n, 3), generator=g) * 0.3).cuda()


@pytest.mark.parametrize("n,d,dtype", [(64, 48, "f32"), (90, 20, "bf16")])
def test_pair(octmc, n, d, dtype):
    log(f"evaluations of a pair after overlapping ones, n={n} d={d} {dtype}")
    S, A, D = _scans(n, d)
    P = octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], dtype=dtype, levels=2)
    m = (n + 1) // 2
    D1 = D[:, ::2, ::2].contiguous()
    want = [x.clone() for l, F in ((0, D), (1, D1)) for x in P.eval(l, F, eta_mode=0)]
    assert D1.shape[1] == m
    _overlap([lambda: P.eval(0, D, eta_mode=0), lambda: P.eval(1, D1, eta_mode=0), lambda: P.eval(0, D, eta_mode=0)])
    got = [x for l, F in ((0, D), (1, D1)) for x in P.eval(l, F, eta_mode=0)]
    torch.cuda.synchronize()
    P.close()
    assert all(torch.equal(a, b) for a, b in zip(want, got))


def test_noalloc(octmc):
    log("eval_noalloc after overlapping calls")
    calls = []
    for n, d in ((64, 48), (40, 60)):
        S, A, D = _scans(n, d)
        v = torch.ones(n, device="cuda")
        eta = torch.ones(1, dtype=torch.float64, device="cuda")
        terms = torch.empty(octmc.NTERMS, dtype=torch.float64, device="cuda")
        grad = torch.empty_like(D)
        calls.append((lambda S=S, A=A, D=D, v=v, eta=eta, terms=terms, grad=grad: octmc.eval_noalloc(
            *S, *A, v, v, D, eta, terms, grad, eta_mode=0), (eta, terms, grad)))
    want = []
    for run, out in calls:
        run()
        torch.cuda.synchronize()
        want += [x.clone() for x in out]
    _overlap([run for run, _ in calls])
    got = []
    for run, out in calls:
        run()
        torch.cuda.synchronize()
        got += [x.clone() for x in out]
    assert all(torch.equal(a, b) for a, b in zip(want, got))


@pytest.mark.parametrize("dtype,count", [("f32", 3), ("f32", 4), ("bf16", 3), ("bf16", 4)])
def test_volumes(octmc, dtype, count):
    log(f"evaluations of {count} volumes after overlapping ones, {dtype}")
    n, d = 48, 40
    S, A, D = _scans(n, d, count)
    M = octmc.Multi(S, [0, 1, 0, 1][:count], enface=A, dtype=dtype, levels=1)
    want = [x.clone() for x in M.eval(0, D, eta_mode=0)]
    _overlap([lambda: M.eval(0, D, eta_mode=0)] * 2)
    got = M.eval(0, D, eta_mode=0)
    torch.cuda.synchronize()
    M.close()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
