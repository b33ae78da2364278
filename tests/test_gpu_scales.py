"""Scales that take W'/s out of fp16's range in a few channels, through the calls that choose their kernel: where a stack of moderate
scales is restored and multiplied, such a one stays with the kernels that put 1/s on the activations.  Whole numbers, bit for bit."""
import pytest

from test_gpu_exact import activations, compare, stack

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn,n,batch,lent", [
    (4096, 4096, 16, 24, True),
    (4096, 4096, 16, 32, True),
    (1024, 4096, 16, 24, False),    # restored through the image's own scratch
    (1024, 8192, 16, 32, False),
    (3136, 2560, 12, 193, False),   # beyond 64 tokens: k_batch
    (1024, 4096, 16, 100, False),   # k_rows
])
def test_restored_only_where_the_dense_weight_is_in_range(out, inn, n, batch, lent):
    import torch
    import paper_2410_23918_amd as B
    scratch = torch.empty(B.dense_bytes(out, inn) if lent else 0, dtype=torch.uint8, device="cuda:0")
    assert B.choose_kernel(out, inn, n, 2048, batch, n, scratch.numel()) == B.KERNEL_MATERIALISE
    # scales of 2^-30, and up to 64 tokens (W' between 16 and 4094 is in question beyond) of 2^-11: W' of 32 is out of range over it
    for small, exponent in (((), 0), ((5, 300, 511, inn - 1), 30), *([((5, 300, 511, inn - 1), 11)] if batch <= 64 else [])):
        ps, w = stack(out, inn, n, 2048, small, exponent)
        assert (w.abs().max() > 65504) == bool(small)
        x = activations(batch, inn, batch, small, min(exponent, 24))
        image_scratch = ps.buf[ps.buf.numel() // 256 * 256 - 2048 * inn * 2:]   # the image's last 2048 x in fp16 values
        used = scratch if lent else image_scratch
        used.fill_(0xff)
        torch.cuda.synchronize()
        if lent:
            compare(ps, w, n, x, lambda y: ps.linear_batched_ws(x, n, scratch, y))
        else:
            compare(ps, w, n, x, lambda y: ps.linear_batched(x, n, y))
        assert bool((used != 0xff).any()) == (not small)   # restored there or not
        del ps, w


@pytest.mark.parametrize("out,inn,n,batch", [(448, 768, 24, 6), (832, 1024, 10, 2), (672, 1792, 24, 5)])
def test_activations_over_their_scales_out_of_fp16_range_where_one_token_kernels_serve_the_batch(out, inn, n, batch):
    """Few tokens, estimated faster through k_rows or restored than through the kernels for one token, which hold x/s in fp32: both x/s
    and W'/s are beyond fp16 in one channel, y is not beyond fp32."""
    import torch
    ps, w = stack(out, inn, n, 2048, (5,))
    x = torch.randn((batch, inn), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(1)).half()
    x[:, 5] = 2.0**-13
    y = ps.linear_batched(x, n, out_dtype=torch.float32)
    want = x.double() @ w.t().contiguous()
    assert ((y.double() - want).abs().amax(dim=1) <= 2e-3 * want.abs().amax(dim=1)).all()   # also false for NaN


def test_a_token_of_its_own_keeps_its_precision():
    """Five tokens through a small stack: four in one launch and one by itself, whose x/s and magnitudes stay in fp32."""
    import torch
    import paper_2410_23918_amd as B
    out, inn, n, batch = 288, 1280, 23, 5
    assert B.choose_kernel(out, inn, n, 64, batch, n) == B.KERNEL_DECODE
    ps, w = stack(out, inn, n, 64)
    x = torch.randn((batch, inn), device="cuda:0", generator=torch.Generator(device="cuda:0").manual_seed(1)).half()
    y = ps.linear_batched(x, n, out_dtype=torch.float32).double()
    want = x.double() @ w.t().contiguous()
    errors = (y - want).norm(dim=1) / want.norm(dim=1)
    assert errors.min() < 1e-6 and errors.max() < 1e-3
