"""k_gemm_64, the dense product's 64 x 64 tile, in both orders of its sums: the bits of the 128 x 128 tiles (options 3 and 4), for row and
token counts that end inside a tile, the shortest row (two steps, fewer than its ring), numbers of steps that leave the ring at each of
its places, and every way of sharing the token tiles among the XCDs (one, two, four)."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn,batch", [
    (32, 256, 1),
    (64, 512, 64),
    (96, 768, 65),
    (1056, 1024, 130),     # seventeen row tiles, three token tiles: shared one way
    (544, 512, 200),       # nine and four: four ways
    (544, 4352, 1000),     # nine and sixteen: four ways
    (640, 1280, 513),
    (8192, 256, 100),      # 32 tiles for an XCD
    (256, 4352, 300),
])
@pytest.mark.parametrize("f32", [False, True])
def test_the_bits_of_the_larger_tiles(out, inn, batch, f32):
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + batch)
    ps = B.PackedStack.empty(out, inn, 1, np.ones(inn, np.float32), max_batch=batch)
    wd = torch.randn((out, inn), generator=g, device="cuda:0").half()
    x = torch.randn((batch, inn), generator=g, device="cuda:0").half()
    y = {}
    try:
        for tile in (3, 4, 5, 6, 0):
            B.set_option(B.OPT_DENSE_TILE, tile)
            y[tile] = torch.full((batch, out), float("nan"), dtype=torch.float32 if f32 else torch.float16, device="cuda:0")
            ps.linear_dense(x, wd, y=y[tile])
            torch.cuda.synchronize()
    finally:
        B.set_option(B.OPT_DENSE_TILE, 0)
    assert torch.isfinite(y[3]).all() and torch.isfinite(y[4]).all()
    assert torch.equal(y[5], y[3]) and torch.equal(y[6], y[4])
    assert torch.equal(y[0], y[6 if inn >= 4096 else 5])   # the library takes it for all of these


@pytest.mark.parametrize("inn", [512, 4352])
def test_row_slabs(inn):
    """1184 rows through a scratch for 1024: the last slab's 160 rows are further apart in y than there are rows in the slab."""
    import torch
    import paper_2410_23918_amd as B
    from test_gpu_exact import stack
    out, n, batch = 1184, 2, 200
    ps, _ = stack(out, inn, n, batch)
    g = torch.Generator(device="cuda:0").manual_seed(inn)
    x = torch.randn((batch, inn), generator=g, device="cuda:0").half()
    want = ps.linear_dense(x, ps.restore_weight(n), out_dtype=torch.float32)
    y = torch.full((batch, out), float("nan"), device="cuda:0")
    ps.linear_materialised(x, n, torch.empty((1024, inn), dtype=torch.float16, device="cuda:0"), y)
    torch.cuda.synchronize()
    assert torch.equal(y, want)
