"""octmc_trim: the device memory kept between objects goes back to the device, and
that of live objects stays."""
import pytest
import torch

import paper_2010_06931_amd as octmc


def test_null_context():
    assert octmc.lib().octmc_trim(None) == -1
    assert "NULL" in octmc.lib().octmc_last_error().decode()


@pytest.mark.gpu
def test_kept_memory_goes_back():
    S = [torch.rand((160, 160, 256), device="cuda") for _ in range(2)]
    A = torch.rand((160, 160), device="cuda")
    D = torch.zeros((2, 160, 160, 3), device="cuda")

    def free():
        torch.cuda.synchronize()
        return torch.cuda.mem_get_info()[0]

    live = octmc.Pair(S[0], S[1], ax=A, ay=A)
    want = [x.clone() for x in live.eval(0, D, eta_mode=0)]
    ctx = octmc.context(0)
    ctx.trim()
    before = free()
    P = octmc.Pair(S[0], S[1], ax=A, ay=A)
    during = free()
    assert before - during > 50 << 20  # two volumes of 25 MB and their coarser levels
    P.close()
    assert free() < before - (40 << 20)  # kept for the next object
    ctx.trim()
    assert before - free() < 8 << 20  # what the runtime itself keeps
    got = live.eval(0, D, eta_mode=0)
    torch.cuda.synchronize()
    assert all(torch.equal(a, b) for a, b in zip(want, got))
    live.close()
    ctx.trim()
