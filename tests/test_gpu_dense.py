"""k_gemm_split, the dense product's 128 x 128 tile for long rows: row and token counts that end inside a tile, odd numbers of tiles in
both directions, the shortest row (four steps, fewer than its ring) and rows that leave the ring at each of its places.  Every element
of y."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn,batch", [
    (32, 256, 1),
    (128, 512, 128),
    (160, 768, 129),
    (1056, 1024, 300),     # nine row tiles, three token tiles
    (640, 1280, 513),
])
@pytest.mark.parametrize("f32", [False, True])
def test_every_output_of_the_split_tile(out, inn, batch, f32):
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + batch)
    ps = B.PackedStack.empty(out, inn, 1, np.ones(inn, np.float32), max_batch=batch)
    wd = torch.randn((out, inn), generator=g, device="cuda:0").half()
    x = torch.randn((batch, inn), generator=g, device="cuda:0").half()
    want = x.double() @ wd.double().t().contiguous()
    size = x.double().abs() @ wd.double().abs().t().contiguous()
    y = torch.full((batch, out), float("nan"), dtype=torch.float32 if f32 else torch.float16, device="cuda:0")
    try:
        B.set_option(B.OPT_DENSE_TILE, 4)
        ps.linear_dense(x, wd, y=y)
        torch.cuda.synchronize()
    finally:
        B.set_option(B.OPT_DENSE_TILE, 0)
    # products of fp16 are exact in fp32; at most 32 + in / 128 + 2 roundings of 2^-24 of the sum of absolute values on the way to one
    # element, and one to fp16
    bound = (34 + inn / 128) * 2.0**-24 * size + (0.0 if f32 else 2.0**-11 * want.abs()) + 2.0**-25
    worst = ((y.double() - want).abs() / bound).max().item()
    print(f"{out}x{inn} batch {batch}: largest error {worst:.3f} of its bound", flush=True)
    assert worst <= 1.0   # also false for an element that was not written (NaN)


def test_a_long_row_takes_it():
    """The order of the sums tells the two 128 x 128 tiles apart."""
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(1)
    # 4224 rows x 800 tokens: 231 tiles, but 36 of them would be one XCD's, which has 32 compute units
    for out, inn, batch, split in ((512, 4096, 256, True), (512, 2048, 256, False), (4224, 4096, 800, False), (4096, 4096, 900, True)):
        ps = B.PackedStack.empty(out, inn, 1, np.ones(inn, np.float32), max_batch=batch)
        wd = torch.randn((out, inn), generator=g, device="cuda:0").half()
        x = torch.randn((batch, inn), generator=g, device="cuda:0").half()
        auto = ps.linear_dense(x, wd, out_dtype=torch.float32).clone()
        forced = {}
        try:
            for tile in (3, 4):
                B.set_option(B.OPT_DENSE_TILE, tile)
                forced[tile] = ps.linear_dense(x, wd, out_dtype=torch.float32).clone()
        finally:
            B.set_option(B.OPT_DENSE_TILE, 0)
        torch.cuda.synchronize()
        assert not torch.equal(forced[3], forced[4])
        assert torch.equal(auto, forced[4 if split else 3])
