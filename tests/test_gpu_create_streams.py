"""Creating an object again, from kept blocks, waits for its own stream only."""
import pytest
import torch

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def octmc():
    import paper_2010_06931_amd as m
    return m


@pytest.mark.parametrize("count", [2, 3])
def test_other_streams_go_on(octmc, count):
    log(f"creation of {count} volumes beside another stream's work")
    S = [torch.rand((40, 40, 48), device="cuda") for _ in range(count)]
    A = [torch.rand((40, 40), device="cuda") for _ in range(count)]

    def create():
        if count == 2:
            return octmc.Pair(S[0], S[1], ax=A[0], ay=A[1], levels=2)
        return octmc.Multi(S, [0, 1, 0], enface=A, levels=2)

    x = torch.zeros((4096, 4096), device="cuda")
    went_on = []
    for _ in range(4):  # two streams may share one of the device's queues
        own, other, done = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Event()
        with torch.cuda.stream(own):
            create().close()
        torch.cuda.synchronize()
        with torch.cuda.stream(other):
            for _ in range(100):
                torch.mm(x, x, out=torch.empty_like(x))  # some 1 ms each
            done.record()
        with torch.cuda.stream(own):
            P = create()
        went_on.append(not done.query())
        torch.cuda.synchronize()
        P.close()
    assert any(went_on)
