"""Whole numbers through every kernel that rebuilds the weight: factors, scales and activations whose magnitudes, sums and outputs are
whole numbers that fp16 and fp32 hold exactly, so that y has to be equal.  No magnitude is zero and no activation is: one lost,
misplaced or repeated sign of one weight in one block changes y."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def stack(out, inn, n, max_batch, small=(), exponent=30):
    """(packed stack, W' over the scales in fp64): odd magnitudes of at most 31, scales 1 and, in the channels `small`, 2^-exponent"""
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + n)
    s = np.ones(inn, np.float32)
    s[list(small)] = 2.0**-exponent
    ps = B.PackedStack.empty(out, inn, n, s, max_batch=max_batch)
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    w = torch.zeros((out, inn), device="cuda:0", dtype=torch.float64)
    for _ in range(n):
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
        u = torch.randint(-1, 2, (out, 16), generator=g, device="cuda:0").half()
        v = 2 * torch.randint(-1, 2, (inn, 16), generator=g, device="cuda:0").half()
        u[:, 0] = v[:, 0] = 1.0
        ps.push_block_device(words, u, v)
        m = u.double() @ v.double().t().contiguous()
        w += torch.where(((words[:, :, None] >> bits) & 1).reshape(out, inn).bool(), m, -m)
    assert w.abs().max() <= 2048   # fp16 holds them
    return ps, w / torch.from_numpy(s).to("cuda:0").double()


def activations(batch, inn, seed, small=(), exponent=24):
    import torch
    g = torch.Generator(device="cuda:0").manual_seed(seed)
    x = torch.randint(1, 5, (batch, inn), generator=g, device="cuda:0") * (2 * torch.randint(0, 2, (batch, inn), generator=g, device="cuda:0") - 1)
    x = x.half()
    for c in small:
        x[:, c] *= 2.0**-exponent
    return x


def compare(ps, w, n, x, call):
    import torch
    want = x.double() @ w.t().contiguous()
    assert (x.double().abs() @ w.abs().t().contiguous()).max() < 2**24   # every partial sum in fp32
    y = torch.full((x.shape[0], w.shape[0]), float("nan"), device="cuda:0")
    for _ in range(2):   # the second call finds the counters as the first left them
        call(y)
        torch.cuda.synchronize()
        assert torch.equal(y.double(), want)


@pytest.mark.parametrize("out,inn,n,batch,tiles", [
    (32, 256, 45, 2, 2), (32, 256, 45, 2, 4),
    (160, 768, 45, 17, 2), (160, 768, 45, 17, 4),       # a ragged second row group, three chunks
    (128, 1280, 60, 33, 2), (128, 1280, 60, 33, 4),     # the columns split
    (416, 2816, 45, 64, 2), (416, 2816, 45, 64, 4),
    (224, 1536, 60, 129, 2), (224, 1536, 60, 129, 4),   # three token groups
    (64, 512, 1, 24, 0), (512, 1024, 2, 8, 0),
    (736, 512, 3, 4, 0), (832, 768, 3, 50, 0),          # k_fused
    (384, 1024, 8, 3, 0),
    (3264, 256, 12, 220, 0), (5312, 1536, 2, 249, 0),   # k_tile, one and three pairs of chunks
    (96, 1280, 7, 1100, 0), (96, 1280, 44, 1100, 0),    # k_tile, k_panel
])
def test_batches(out, inn, n, batch, tiles):
    import paper_2410_23918_amd as B
    ps, w = stack(out, inn, n, max(64, batch))
    x = activations(batch, inn, batch)
    B.set_option(B.OPT_BATCH_TILES, tiles)
    try:
        compare(ps, w, n, x, lambda y: ps.linear_batched(x, n, y=y, kernel=B.KERNEL_PANEL))
    finally:
        B.set_option(B.OPT_BATCH_TILES, 0)


@pytest.mark.parametrize("out,inn,n,batch", [
    (1056, 1024, 3, 31), (64, 2048, 2, 31),              # k_fused, two and four pairs of chunks
    (1056, 1024, 8, 4), (1056, 2048, 8, 4),              # its columns split two and four ways
    (64, 4096, 8, 3), (1056, 2048, 6, 31),               # eight ways; 24 steps
    (32, 256, 45, 65), (96, 512, 32, 128),               # k_panel, one tile of 128 tokens
    (64, 256, 32, 129), (96, 512, 45, 256),              # two
])
def test_batches_without_k_rows(out, inn, n, batch):
    """Matrices of few rows through the kernels that serve the larger ones, which take seconds to make and to check"""
    import paper_2410_23918_amd as B
    ps, w = stack(out, inn, n, max(64, batch))
    x = activations(batch, inn, batch)
    B.set_option(B.OPT_ROWS_CHUNKS, 16)
    try:
        compare(ps, w, n, x, lambda y: ps.linear_batched(x, n, y=y, kernel=B.KERNEL_PANEL))
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)


@pytest.mark.parametrize("tiles", [2, 4])
@pytest.mark.parametrize("batch", [2, 17, 64, 130])
def test_scales_out_of_fp16_range(batch, tiles):
    """W'/s beyond fp16's largest value in four channels: k_batch starts over with 1/s on the activations."""
    import paper_2410_23918_amd as B
    small = (5, 300, 511, 1279)
    ps, w = stack(96, 1280, 45, max(64, batch), small)
    x = activations(batch, 1280, batch, small)
    B.set_option(B.OPT_BATCH_TILES, tiles)
    try:
        compare(ps, w, 45, x, lambda y: ps.linear_batched(x, 45, y=y, kernel=B.KERNEL_PANEL))
    finally:
        B.set_option(B.OPT_BATCH_TILES, 0)


@pytest.mark.parametrize("out,inn,n", [(32, 256, 1), (64, 256, 9), (1056, 2304, 3), (512, 512, 4), (32, 14336, 20)])
def test_one_token(out, inn, n):
    ps, w = stack(out, inn, n, 1)
    x = activations(1, inn, n)
    compare(ps, w, n, x, lambda y: ps.linear_batched(x, n, y=y))


@pytest.mark.parametrize("out,inn,n", [(32, 256, 1), (96, 512, 2), (160, 1280, 5), (1056, 768, 29), (17408, 2048, 3)])
def test_restored_weight(out, inn, n):
    import torch
    ps, w = stack(out, inn, n, 1)
    got = torch.full((out, inn), float("nan"), dtype=torch.float16, device="cuda:0")
    ps.restore_weight(n, got)
    torch.cuda.synchronize()
    assert torch.equal(got.double(), w)
