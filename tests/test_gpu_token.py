"""k_token, the kernel for one token through a small stack: fewer units than wavefronts, exactly as many and one more, one workgroup
per row tile and many (the last one to arrive adds their rows, in more than one round from 65 on), activations and scales far apart,
few activations.  Every element of y."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


SHAPES = [
    (32, 256, 1),       # one unit: seven wavefronts without
    (64, 256, 8),       # eight: one each
    (64, 256, 9),       # a second workgroup with one unit
    (96, 768, 5),
    (1056, 2304, 3),
    (512, 512, 4),
    (32, 14336, 20),    # 140 workgroups per row tile
]


def check(out, inn, n, s, x, v_scale, silent=()):
    """Blocks with V of block i times v_scale[i] and zero in the channels `silent`; fp32 and fp16 outputs of one token, three calls
    each (a later call finds the counters as the one before left them)."""
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(out + inn + n)
    ps = B.PackedStack.empty(out, inn, n, s)
    xs = x.double() * torch.from_numpy(1.0 / s.astype(np.float64)).to("cuda:0")
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    want = torch.zeros(out, device="cuda:0", dtype=torch.float64)
    size = torch.zeros_like(want)
    for i in range(n):
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
        u = (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half()
        v = (v_scale[i] * torch.randn((inn, 16), generator=g, device="cuda:0")).half()
        v[list(silent)] = 0.0
        ps.push_block_device(words, u, v)
        m = u.double() @ v.double().t().contiguous()
        want += torch.where(((words[:, :, None] >> bits) & 1).reshape(out, inn).bool(), m, -m) @ xs
        size += u.double().abs() @ (v.double().abs().t().contiguous() @ xs.abs())
    # fp32 throughout: 1/s, x/s, 16 ranks in the matrix product, 32 multiply-adds and 4 additions per lane, the two lane halves, 8
    # wavefronts, the partial rows of the workgroups (every 16th in turn, then 16); a rounding is at most 2^-23 (the matrix
    # product's may cut off) of the sum of absolute values
    parts = (n * inn // 256 + 7) // 8
    bound32 = (2 + 16 + 32 + 4 + 1 + 8 + (parts / 16 + 17 if parts > 1 else 0)) * 2.0**-23 * size
    for dtype, bound in ((torch.float32, bound32 + 1e-30), (torch.float16, bound32 + 2.0**-11 * want.abs() + 2.0**-25)):
        for _ in range(3):
            y = torch.full((1, out), float("nan"), dtype=dtype, device="cuda:0")
            ps.linear_batched(x[None], n, y)
            torch.cuda.synchronize()
            worst = ((y[0].double() - want).abs() / bound).max().item()
            print(f"{out}x{inn} n={n} {dtype}: largest error {worst:.3f} of its bound", flush=True)
            assert worst <= 1.0   # also false for an element that was not written (NaN)


@pytest.mark.parametrize("out,inn,n", SHAPES)
@pytest.mark.parametrize("wide", [False, True])
def test_every_output_of_a_small_stack(out, inn, n, wide):
    import torch
    s = np.exp((3.0 if wide else 0.5) * np.random.default_rng(n).standard_normal(inn)).astype(np.float32)
    x = torch.randn((inn,), generator=torch.Generator(device="cuda:0").manual_seed(n), device="cuda:0").half()
    if wide:
        x *= 2.0**-8   # |y| below fp16's largest value
    check(out, inn, n, s, x, [4.0 if wide and i == 0 else 0.02 for i in range(n)])


@pytest.mark.parametrize("scale", [1e-8, 1e-10, 1e-12])
@pytest.mark.parametrize("out,inn,n", [(512, 512, 4), (96, 768, 5)])
def test_a_channel_scaled_far_down_with_no_weight(out, inn, n, scale):
    """V follows the scales: the channel's x/s is the largest by far, and none of it reaches y."""
    import torch
    s = np.exp(0.5 * np.random.default_rng(n).standard_normal(inn)).astype(np.float32)
    silent = (3, inn - 200)
    s[list(silent)] = scale
    x = torch.randn((inn,), generator=torch.Generator(device="cuda:0").manual_seed(n), device="cuda:0").half()
    check(out, inn, n, s, x, [0.1] * n, silent)


@pytest.mark.parametrize("hot", [1, 8, 40])
def test_few_activations(hot):
    """One column, or a few, of the weight: no other rounding hides how exactly a product is taken."""
    import torch
    out, inn, n = 512, 512, 4
    s = np.exp(0.5 * np.random.default_rng(n).standard_normal(inn)).astype(np.float32)
    g = torch.Generator(device="cuda:0").manual_seed(hot)
    x = torch.zeros((inn,), dtype=torch.float16, device="cuda:0")
    x[torch.randperm(inn, generator=g, device="cuda:0")[:hot]] = torch.randn((hot,), generator=g, device="cuda:0").half()
    check(out, inn, n, s, x, [0.1] * n)


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


@pytest.mark.parametrize("inn,shapes,token", [
    (1024, ((160, 3), (64, 2), (1056, 1)), True),
    (2048, ((96, 9), (1024, 2)), True),
    (4096, ((1024, 9), (4096, 9)), False),                   # the first alone is k_token's
    (12288, ((256, 5), (320, 5), (1312, 1)), False),         # 786 workgroups: 14.7 us, through k_decode 12.0
])
def test_merged_launches(inn, shapes, token):
    """A launch has one kernel for all its stacks: every output against fp64 and against the stack's own launch, which may be the
    other kernel's."""
    import torch
    import paper_2410_23918_amd as B
    g = torch.Generator(device="cuda:0").manual_seed(inn)
    x = torch.randn((inn,), generator=g, device="cuda:0").half()
    bits = torch.arange(32, device="cuda:0", dtype=torch.int32)
    items, wants = [], []
    for out, n in shapes:
        ps = B.PackedStack.empty(out, inn, n, np.ones(inn, np.float32))
        want = torch.zeros(out, device="cuda:0", dtype=torch.float64)
        for _ in range(n):
            words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device="cuda:0", dtype=torch.int64).to(torch.int32)
            u = (0.1 * torch.randn((out, 16), generator=g, device="cuda:0")).half()
            v = (0.1 * torch.randn((inn, 16), generator=g, device="cuda:0")).half()
            ps.push_block_device(words, u, v)
            m = u.double() @ v.double().t().contiguous()
            want += torch.where(((words[:, :, None] >> bits) & 1).reshape(out, inn).bool(), m, -m) @ x.double()
        items.append((x, ps, n, torch.full((out,), float("nan"), dtype=torch.float16, device="cuda:0")))
        wants.append(want)
    plan = B.TokenPlan(B.make_jobs(items))
    assert plan.steps == 1
    plan.launch()
    got = [y.clone() for *_, y in items]
    single = [ps.linear(x, n).clone() for _, ps, n, _ in items]
    B.set_option(B.OPT_DECODE_EARLY, 3)   # what k_decode takes by itself
    try:
        B.TokenPlan(B.make_jobs(items)).launch()
        torch.cuda.synchronize()
    finally:
        B.set_option(B.OPT_DECODE_EARLY, 0)
    assert all(torch.equal(a, y) for a, (*_, y) in zip(got, items)) != token
    for a, b, want in zip(got, single, wants):
        # either kernel's error is 2e-3 of the largest output at most
        assert (a.double() - want).abs().max() <= 2e-3 * want.abs().max()
        assert (a.double() - b.double()).abs().max() <= 2e-3 * want.abs().max()
