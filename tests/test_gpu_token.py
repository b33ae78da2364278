"""k_token, the kernel for one token through a small stack: fewer units than wavefronts, exactly as many and one more, one workgroup
per row tile and many (the last one to arrive adds their rows, in more than one round from 65 on), activations and scales far apart.
Every element of y."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("out,inn,n", [
    (32, 256, 1),       # one unit: seven wavefronts without
    (64, 256, 8),       # eight: one each
    (64, 256, 9),       # a second workgroup with one unit
    (96, 768, 5),
    (1056, 2304, 3),
    (512, 512, 4),
    (32, 14336, 20),    # 140 workgroups per row tile
])
@pytest.mark.parametrize("wide", [False, True])
def test_every_output_of_a_small_stack(out, inn, n, wide):
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + n)
    s = np.exp((3.0 if wide else 0.5) * np.random.default_rng(n).standard_normal(inn)).astype(np.float32)
    ps = B.PackedStack.empty(out, inn, n, s)
    x = torch.randn((inn,), generator=g, device="cuda:0").half()
    if wide:
        x *= 2.0**-8   # |y| below fp16's largest value
    xs = x.double() * torch.from_numpy(1.0 / s).to("cuda:0").double()
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    want = torch.zeros(out, device="cuda:0", dtype=torch.float64)
    size = torch.zeros_like(want)
    floor = torch.zeros_like(want)
    for i in range(n):
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
        u = (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half()
        v = ((4.0 if wide and i == 0 else 0.02) * torch.randn((inn, 16), generator=g, device="cuda:0")).half()
        ps.push_block_device(words, u, v)
        m = u.double() @ v.double().t().contiguous()
        want += torch.where(((words[:, :, None] >> bits) & 1).reshape(out, inn).bool(), m, -m) @ xs
        size += u.double().abs() @ (v.double().abs().t().contiguous() @ xs.abs())
        # half a unit of fp16's subnormals for x/s and for its product with V, both at a scale that puts the largest product of a
        # chunk (V taken as 1 at least) above 2^13
        top = (v.double().abs().amax(dim=1).view(-1, 256).amax(dim=1).clamp(min=1.0) * xs.abs().view(-1, 256).amax(dim=1)) * 2.0**-13
        floor += u.double().abs().sum(dim=1) * (top[:, None] * 2.0**-25 * (1.0 + v.double().abs().amax(dim=1).view(-1, 256))).sum()
    # x/s and its product with V rounded to 11 bits (2^-11 each), sums of 16-rank products in fp32, y rounded to fp16
    bound = (2.0**-10 * 1.01 + (inn / 16 + 64) * 2.0**-24) * size + floor + 2.0**-11 * want.abs() + 2.0**-25
    y = torch.full((out,), float("nan"), dtype=torch.float16, device="cuda:0")
    for _ in range(3):   # a later call finds the counters as the one before left them
        y.fill_(float("nan"))
        ps.linear(x, n, y)
        torch.cuda.synchronize()
        worst = ((y.double() - want).abs() / bound).max().item()
        print(f"{out}x{inn} n={n}: largest error {worst:.3f} of its bound", flush=True)
        assert worst <= 1.0   # also false for an element that was not written (NaN)


def test_it_is_the_kernel_taken():
    """A forced work split goes to the other kernel, whose fixed point gives other last bits."""
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(5)
    for out, inn, n, small in ((512, 512, 4, True), (1024, 4096, 3, True), (4096, 4096, 16, False)):
        ps = B.PackedStack.empty(out, inn, n, np.ones(inn, np.float32))
        for _ in range(n):
            ps.push_block_device(torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32),
                                 (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half(),
                                 (0.1 * torch.randn((inn, 16), generator=g, device="cuda:0")).half())
        x = torch.randn((inn,), generator=g, device="cuda:0").half()
        auto = ps.linear(x, n).clone()
        try:
            B.set_option(B.OPT_DECODE_EARLY, 3)   # what k_decode takes by itself
            forced = ps.linear(x, n).clone()
        finally:
            B.set_option(B.OPT_DECODE_EARLY, 0)
        torch.cuda.synchronize()
        assert torch.equal(auto, forced) != small
        assert (auto.float() - forced.float()).norm() < 2e-3 * forced.float().norm()


@pytest.mark.parametrize("bad", [float("inf"), float("nan")])
def test_what_is_not_finite_stays_so(bad):
    import torch
    import paper_2410_23918_amd as B
    ps = B.PackedStack.empty(64, 512, 2, np.ones(512, np.float32))
    g = torch.Generator(device="cuda:0").manual_seed(6)
    for _ in range(2):
        ps.push_block_device(torch.full((64, 16), -1, dtype=torch.int32, device="cuda:0"),
                             torch.full((64, 16), 0.25, dtype=torch.float16, device="cuda:0"),
                             torch.full((512, 16), 0.25, dtype=torch.float16, device="cuda:0"))
    x = torch.randn((512,), generator=g, device="cuda:0").half()
    x[300] = bad
    y = ps.linear(x, 2)
    assert not torch.isfinite(y).any()
    assert not ps.linear(torch.zeros_like(x), 2).any()
