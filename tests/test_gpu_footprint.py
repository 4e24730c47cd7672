"""A served request uses what was reserved for it: all of it with inputs on the host,
and all but the room of the structural inputs' copies with inputs on the device."""
import ctypes as C

import pytest
import torch

from gpu_util import log

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("host", [True, False])
@pytest.mark.parametrize("n,d,dtype,levels,given,flags,merged", [
    (24, 33, "f32", 3, ("enface",), 0, False), (24, 33, "bf16", 3, ("octa", "valid"), 0, True),
    (32, 40, "f32", 2, ("octa",), "detect project", True), (20, 21, "f16", 1, ("octa", "enface"), "project", True),
    (40, 48, "f32", 0, ("octa", "enface", "valid"), "detect", False)])
def test_used_as_reserved(host, n, d, dtype, levels, given, flags, merged):
    import paper_2010_06931_amd as octmc
    log(f"served request n={n} d={d} {dtype} {given} {flags} host={host}")
    L = octmc.lib()
    where = "cpu" if host else "cuda"
    r = octmc.Request()
    L.octmc_params_default(C.byref(r.params))
    r.params.levels, r.params.iters_per_level = levels, 2
    for f, v in (("detect", octmc.DETECT_INVALID), ("project", octmc.ENFACE_PROJECT)):
        if flags and f in flags:
            r.params.flags |= v
    r.shape = octmc.Shape(n, n, d, {"f32": 0, "bf16": 1, "f16": 2}[dtype], octmc.MEM_HOST if host else octmc.MEM_DEVICE)
    keep = {"oct": [torch.rand((n, n, d), device=where) for _ in range(2)]}
    if "octa" in given:
        keep["octa"] = [torch.rand((n, n, d), device=where) for _ in range(2)]
    if "enface" in given:
        keep["enface"] = [torch.rand((n, n), device=where) for _ in range(2)]
    if "valid" in given:
        keep["valid"] = [torch.ones(n, device=where) for _ in range(2)]
        keep["valid"][0][3] = 0.0
    for k, v in keep.items():
        setattr(r, k + "_x", v[0].data_ptr())
        setattr(r, k + "_y", v[1].data_ptr())
    disp, out = torch.empty((2, n, n, 3), device="cuda"), torch.empty((n, n, d), device="cuda")
    r.disp_out = disp.data_ptr()
    if merged:
        r.merged_oct = out.data_ptr()
    torch.cuda.synchronize()
    srv = octmc.Server(1 << 30, max_active=1)
    octmc._check(L.octmc_server_submit(srv._h, C.byref(r), None))
    (c,) = srv.poll(1, wait_ms=60000)
    srv.close()
    assert c["status"] == 0, c["error"]
    room = 0 if host else 2 * ((n * n * d * 4 + 255) // 256 * 256)
    assert c["bytes_reserved"] - c["bytes_used"] == room, c
