"""The decomposition reads nothing from its workspace that it has not written: the same bits whatever the workspace held, for numbers of
parts of the Gram matrix (128 rows each up to 64 parts) below, at and above the 16 and 32 that are loaded at a time, on either side."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn", [(32, 256), (512, 512), (160, 4096), (4096, 512), (4224, 256), (2112, 2304)])
def test_the_workspace_may_hold_anything(out, inn):
    import torch
    import paper_2410_23918_amd as B
    from paper_2410_23918_amd.binding import _check, lib
    g = torch.Generator(device="cuda:0").manual_seed(out + inn)
    w = 0.02 * torch.randn((out, inn), generator=g, device="cuda:0")
    s = np.ones(inn, np.float32)
    size = lib().bitstack_decompose_workspace_bytes(out, inn, 16)
    results = []
    for fill in (0x00, 0xff, 0x40):   # zeros; NaN; 32.5 as fp64
        ws = torch.full((size,), fill, dtype=torch.uint8, device="cuda:0")
        sw = torch.empty((2, out, inn // 32), dtype=torch.int32, device="cuda:0")
        u = torch.empty((2, out, 16), dtype=torch.float16, device="cuda:0")
        v = torch.empty((2, inn, 16), dtype=torch.float16, device="cuda:0")
        _check(lib().bitstack_decompose(w.data_ptr(), s.ctypes.data, out, inn, 16, 2, 4, sw.data_ptr(), u.data_ptr(), v.data_ptr(),
                                        ws.data_ptr(), size, torch.cuda.current_stream().cuda_stream), "bitstack_decompose")
        torch.cuda.synchronize()
        assert torch.isfinite(u).all() and torch.isfinite(v).all()
        results.append((sw, u, v))
    for other in results[1:]:
        for a, b in zip(results[0], other):
            assert torch.equal(a, b)
