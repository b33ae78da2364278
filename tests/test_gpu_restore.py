"""The restore kernel at the edges of its tiling: row counts that end inside a row tile's workgroup, one and several column
chunks, one block and more (the pipeline runs three steps ahead), several row groups per workgroup.  Every element
against Eq. 8 in fp64 on the device."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn,n", [
    (32, 256, 1),        # one wavefront with rows, one step
    (96, 512, 2),
    (128, 256, 3),
    (160, 1280, 5),      # a second, almost empty row group; the ring of four buffers wraps
    (1056, 768, 29),     # the largest number of blocks
    (49280, 2048, 2),    # 386 row groups x 8 chunks: two row groups per workgroup, the last one ragged
])
def test_every_element_of_the_restored_weight(out, inn, n):
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + n)
    s = np.exp(0.5 * np.random.default_rng(n).standard_normal(inn)).astype(np.float32)
    ps = B.PackedStack.empty(out, inn, n, s)
    w = torch.zeros((out, inn), device="cuda:0", dtype=torch.float64)
    mag = torch.zeros((out, inn), device="cuda:0")   # sum over blocks of |U| |V|^T
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    for _ in range(n):
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
        u = (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half()
        v = (0.1 * torch.randn((inn, 16), generator=g, device="cuda:0")).half()
        ps.push_block_device(words, u, v)
        m = u.double() @ v.double().t().contiguous()
        for r in range(0, out, 4096):
            plus = ((words[r:r + 4096, :, None] >> bits) & 1).reshape(-1, inn).bool()
            w[r:r + 4096] += torch.where(plus, m[r:r + 4096], -m[r:r + 4096])
        mag += u.float().abs() @ v.float().abs().t().contiguous()
    rs = torch.from_numpy(1.0 / s).to("cuda:0")
    w *= rs
    mag *= rs
    got = torch.full((out, inn), float("nan"), dtype=torch.float16, device="cuda:0")
    ps.restore_weight(n, got)
    torch.cuda.synchronize()
    # n blocks of 16 ranks added in fp32 (at most n + 16 roundings of 2^-23 of the sum of absolute values; a matrix product may cut
    # off) and times 1/s, rounded to fp16 once: 2^-11 of it, or half the spacing of subnormals
    bound = 2.0**-11 * w.abs() * 1.01 + (n + 16) * 2.0**-23 * mag + 2.0**-25
    worst = ((got.double() - w).abs() / bound).max().item()
    print(f"{out}x{inn} n={n}: largest error {worst:.2f} of its bound", flush=True)
    assert worst <= 1.0   # also false for an element that was not written (NaN)
