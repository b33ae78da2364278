"""The choice between the batch kernels and restoring beyond 64 tokens: shapes where the two are far apart, timed both ways on MI355X
(microseconds, batch kernels / restoring and multiplying)."""
import pytest

BIG = 1 << 40


@pytest.mark.parametrize("out,inn,n,tokens,scratch,restore", [
    (768, 14080, 13, 82, BIG, False),      # few rows: 46 / 104
    (6368, 3072, 1, 121, BIG, False),      # one block: 19 / 41
    (4096, 4096, 16, 256, BIG, True),      # 93 / 50
    (2528, 5888, 1, 298, 0, False),        # in slabs through the image's own scratch, the second of 480 rows: 33 / 99
    (2688, 13568, 9, 78, 0, False),        # 77 / 211
    (28672, 8192, 16, 2048, 0, True),      # 2100 / 1350
    # more than 1024 tokens through few rows: k_tile, not k_rows, is what restoring is compared with
    (544, 14336, 2, 1800, BIG, True),      # 245 / 99
    (512, 2048, 1, 2048, BIG, True),       # 44 / 18
    (512, 2048, 1, 2048, 0, True),         # 44 / 18
    (544, 14336, 2, 1800, 0, True),        # 245 / 98
])
def test_far_from_the_crossover(out, inn, n, tokens, scratch, restore):
    import paper_2410_23918_amd as B
    got = B.choose_kernel(out, inn, n, 2048, tokens, n, scratch)
    assert got == (B.KERNEL_MATERIALISE if restore else B.KERNEL_PANEL)


@pytest.mark.parametrize("out,inn,n,max_batch,scratch", [(288, 1280, 23, 64, 0), (480, 1280, 24, 2048, 0), (416, 1280, 24, 64, BIG)])
def test_five_tokens_of_which_one_is_a_launch_of_its_own(out, inn, n, max_batch, scratch):
    """Estimated faster through k_rows or restored, but that token would be rounded to fp16 on its way (tests/test_gpu_scales.py); 19 us, 28
    and 29 with k_rows."""
    import paper_2410_23918_amd as B
    assert B.choose_kernel(out, inn, n, max_batch, 5, n, scratch) == B.KERNEL_DECODE
