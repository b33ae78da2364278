"""The batch kernel for up to 64 tokens at the edges of its tiling: row counts that end inside a workgroup, chunk counts that
leave teams without a chunk, both sides of its 16- and 32-token groups, with and without a column split (whose partial
tiles meet in the workspace).  45 blocks: more than the other small-batch kernel holds, so this one runs; the cases of one
and two blocks are among those that are seen to take it.  Matrices of few rows go to k_rows instead: every list runs without it (this kernel) and
as the library chooses.  Every element of y in fp32."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu

without_and_with_rows = pytest.mark.parametrize("rows", [16, 0])   # OPT_ROWS_CHUNKS: never, the library's choice


@pytest.mark.parametrize("out,inn", [
    (32, 256),       # one row tile, one chunk: three of four teams idle
    (96, 1280),      # 5 chunks: split over workgroups
    (160, 2816),     # 11 chunks, a ragged second row group
])
@pytest.mark.parametrize("batch", [2, 16, 17, 32, 33, 64])
@without_and_with_rows
def test_every_output_of_the_small_batch_kernel(out, inn, batch, rows):
    check(out, inn, 45, batch, rows=rows)


@pytest.mark.parametrize("inn,batch", [(8192, 1), (8192, 2), (8192, 33), (7168, 16), (5120, 17)])
@without_and_with_rows
def test_many_column_ranges(inn, batch, rows):
    """32, 28 and 20 column chunks in eight, seven and five ranges: the last workgroup to arrive adds that many partial tiles."""
    check(32, inn, 45, batch, rows=rows)


# one block (a step of the ring, then the activations and the next scales at once) and two, in one and two chunk iterations
FEW_BLOCKS = [(448, 256, 1, 16), (96, 1024, 1, 32), (64, 512, 1, 24), (512, 1024, 2, 8), (512, 1024, 2, 24), (9056, 2048, 1, 20),
              (14336, 2048, 2, 8), (9056, 1280, 2, 60)]


@pytest.mark.parametrize("out,inn,n,batch", FEW_BLOCKS)
@without_and_with_rows
def test_few_blocks(out, inn, n, batch, rows):
    check(out, inn, n, batch, rows=rows)


@pytest.mark.parametrize("out,inn,n", [
    (96, 1280, 60),    # enough workspace to split the columns of several token groups
    (160, 2816, 12),
])
@pytest.mark.parametrize("batch", [65, 128, 129, 1000, 1024, 1025])
@without_and_with_rows
def test_more_than_64_tokens_in_groups(out, inn, n, batch, rows):
    """Both sides of the 64-token groups, and of the 1024 tokens up to which they are taken."""
    check(out, inn, n, batch, rows=rows)


@pytest.mark.parametrize("batch", [2, 17, 64, 130])
@without_and_with_rows
def test_weights_over_their_scales_out_of_fp16_range(batch, rows):
    """Four channels scaled down by 2^-30 whose activations are tiny or zero: a weight over its scale is beyond fp16's largest value
    there (W' is of the order of 0.2), the activation over the scale is not."""
    check(96, 1280, 45, batch, small=(5, 300, 511, 1279), rows=rows)


@pytest.mark.parametrize("out,inn,n,batch,fused", [
    (736, 512, 3, 4, True),       # three steps: 6.7 us, k_batch 8.7
    (5376, 512, 3, 16, True),     # 7.0, 9.2
    (96, 512, 2, 30, True),       # two steps: 7.4, 8.7
    (832, 768, 3, 50, True),      # six steps, two token groups: 9.7, 11.7
    (384, 1024, 8, 3, True),      # eight steps, two column ranges: 12.5, 14.2
    (448, 256, 1, 4, False),      # one step: 8.0, 6.7
    (4096, 4096, 16, 16, False),
    *((*c, False) for c in FEW_BLOCKS),
])
def test_the_kernel_taken_for_few_steps(out, inn, n, batch, fused):
    """k_fused rounds x/s to fp16, k_batch W'/s: with weights n, scales 7 and activations 7 the one is exact, the other is not."""
    import torch
    import paper_2410_23918_amd as B
    ps = B.PackedStack.empty(out, inn, n, np.full(inn, 7.0, np.float32), max_batch=64)
    for _ in range(n):
        ps.push_block_device(torch.full((out, inn // 32), -1, dtype=torch.int32, device="cuda:0"),
                             torch.full((out, 16), 0.25, dtype=torch.float16, device="cuda:0"),
                             torch.full((inn, 16), 0.25, dtype=torch.float16, device="cuda:0"))
    y = torch.full((batch, out), float("nan"), device="cuda:0")
    ps.linear_batched(torch.full((batch, inn), 7.0, dtype=torch.float16, device="cuda:0"), n, y=y, kernel=B.KERNEL_PANEL)
    want = float(n * inn if fused else torch.tensor(n / 7.0).half()) * (1 if fused else 7 * inn)
    # the sums are of equal numbers: exact for k_fused, for k_batch within fp32's rounding of in / 16 + 16 additions
    assert (y - want).abs().max().item() <= (0.0 if fused else (inn / 16 + 16) * 2.0**-24 * want)


@pytest.mark.parametrize("out,inn,n,batch,tile", [
    (3264, 256, 12, 220, True),    # one column chunk: 21.9 us, k_batch 24.7
    (5312, 1536, 2, 249, True),    # estimates within 1 %: 30.7, 35.2
    (11424, 768, 5, 78, True),     # 27.7, 30.0
    (864, 256, 9, 124, False),     # 19.4, 19.2
    (768, 12032, 18, 84, False),   # 410, 57
])
def test_the_kernel_taken_beyond_64_tokens(out, inn, n, batch, tile):
    """k_tile rearranges the activations in the image's scratch, k_batch reads them where they are."""
    import torch
    import paper_2410_23918_amd as B
    ps = B.PackedStack.empty(out, inn, n, np.full(inn, 7.0, np.float32), max_batch=1024)
    for _ in range(n):
        ps.push_block_device(torch.full((out, inn // 32), -1, dtype=torch.int32, device="cuda:0"),
                             torch.full((out, 16), 0.25, dtype=torch.float16, device="cuda:0"),
                             torch.full((inn, 16), 0.25, dtype=torch.float16, device="cuda:0"))
    torch.cuda.synchronize()
    end = ps.buf.numel() // 256 * 256
    scratch = ps.buf[end - 1024 * inn * 2:end]   # the image's last 1024 x in fp16 values
    scratch.zero_()
    ps.linear_batched(torch.full((batch, inn), 7.0, dtype=torch.float16, device="cuda:0"), n, kernel=B.KERNEL_PANEL)
    assert bool(scratch.any()) == tile


@without_and_with_rows
def test_an_infinite_activation_stays_with_its_token(rows):
    check(96, 1280, 45, 20, infinite=7, rows=rows)


def check(out, inn, n, batch, small=(), infinite=None, rows=0):
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + batch)
    s = np.exp(0.5 * np.random.default_rng(batch).standard_normal(inn)).astype(np.float32)
    s[list(small)] = 2.0**-30
    ps = B.PackedStack.empty(out, inn, n, s, max_batch=max(64, batch))
    w = torch.zeros((out, inn), device="cuda:0", dtype=torch.float64)
    mag = torch.zeros_like(w)   # sum over blocks of |U| |V|^T
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    for _ in range(n):
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
        u = (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half()
        v = (0.1 * torch.randn((inn, 16), generator=g, device="cuda:0")).half()
        ps.push_block_device(words, u, v)
        m = u.double() @ v.double().t().contiguous()
        w += torch.where(((words[:, :, None] >> bits) & 1).reshape(out, inn).bool(), m, -m)
        mag += u.double().abs() @ v.double().abs().t().contiguous()
    rs = torch.from_numpy(1.0 / s).to("cuda:0").double()
    w *= rs
    mag *= rs
    x = torch.randn((batch, inn), generator=g, device="cuda:0").half()
    for k, c in enumerate(small):
        x[:, c] = 0.0 if k % 2 else 2.0**-24 * torch.randint(-3, 4, (batch,), generator=g, device="cuda:0").half()
    if infinite is not None:
        x[infinite, 100] = float("inf")
    finite = torch.isfinite(x).all(dim=1)
    y = torch.full((batch, out), float("nan"), device="cuda:0")
    for _ in range(2):   # the second call finds the counters as the first left them
        B.set_option(B.OPT_ROWS_CHUNKS, rows)
        try:
            ps.linear_batched(x, n, y=y, kernel=B.KERNEL_PANEL)
        finally:
            B.set_option(B.OPT_ROWS_CHUNKS, 0)
        torch.cuda.synchronize()
        assert not torch.isfinite(y[~finite]).any()
        xa = x[finite].float().abs().double()
        want = x[finite].double() @ w.t().contiguous()
        # a weight: n blocks of 16 ranks added in fp32 (at most n + 16 roundings of 2^-23 of the sum of absolute values; a matrix product
        # may cut off), times 1/s, rounded to fp16 once (2^-11 of it, or half the spacing of subnormals); then fp32 sums of 16-column
        # products: at most in / 16 + 16 roundings of 2^-24 of the sum of absolute values
        werr = 2.0**-11 * w.abs() * 1.01 + (n + 16) * 2.0**-23 * mag + 2.0**-25
        bound = xa @ werr.t().contiguous() + (inn / 16 + 16) * 2.0**-24 * (xa @ w.abs().t().contiguous())
        if small or infinite is not None or (batch > 1024 and n > 29):
            # 1/s may be on the activations instead (always in the kernel for many tokens and tall stacks): x/s rounded to fp16 (2^-11 of it, or half the spacing of subnormals) and the sum
            # of the magnitudes rounded before the scale (2^-11 of it is in werr, half a subnormal spacing is not)
            wp, xs = (w / rs).abs(), xa * rs
            bound += (2.0**-11 * xs + 2.0**-25) @ wp.t().contiguous() + 2.0**-25 * xs.sum(dim=1, keepdim=True)
        worst = ((y[finite].double() - want).abs() / bound).max().item()
        print(f"{out}x{inn} batch {batch}: largest error {worst:.3f} of its bound", flush=True)
        assert worst <= 1.0   # also false for an element that was not written (NaN)


@pytest.mark.parametrize("tiles", [2, 4])
@pytest.mark.parametrize("out,inn,n,batch", [
    (32, 256, 45, 2),       # one of four row tiles, one of two teams with a chunk
    (160, 768, 45, 17),     # a ragged second row group, three chunks: the second team's last one is none
    (128, 1280, 60, 33),    # the columns split
    (416, 2816, 45, 64),
    (224, 1536, 60, 129),   # three token groups
])
def test_both_numbers_of_row_tiles_per_workgroup(tiles, out, inn, n, batch):
    import paper_2410_23918_amd as B
    B.set_option(B.OPT_BATCH_TILES, tiles)
    try:
        check(out, inn, n, batch)
    finally:
        B.set_option(B.OPT_BATCH_TILES, 0)
