"""k_rows, the batch kernel of one row tile per workgroup: every share of its eight wavefronts between column chunks and blocks, for row
tiles, chunks and blocks that do not divide evenly, as many blocks as groups of them, one chunk, and token counts at the edges of its groups of
32.  A share is taken only if it leaves no group of blocks empty (8 / chunks <= blocks): others are left out.  Every element of y against an
evaluation in 64 bits, and whole numbers bit for bit."""
import numpy as np
import pytest

from oracle import bitstack_oracle as O
from _cases import acts, synth_stack
from test_gpu_exact import activations, compare, stack

pytestmark = pytest.mark.gpu


def shares(stacks):
    """(chunks at a time, *stack) for every share that the stack's blocks allow"""
    return [(c, *s) for s in stacks for c in (1, 2, 4, 8) if 8 // c <= s[2]]


@pytest.mark.parametrize("chunks,out,inn,n", shares([(32, 256, 1), (96, 512, 2), (160, 768, 3), (64, 1280, 5), (352, 2304, 8), (1056, 2048, 9)]))
def test_every_output_of_every_share(chunks, out, inn, n):
    import torch
    import paper_2410_23918_amd as B
    st = synth_stack(3, out, inn, n, tag=17)
    ps = B.PackedStack(st.sign_words(), st.U, st.V, st.s, max_batch=200)
    x = acts(3, 200, inn, tag=17)
    ref = O.forward_dense(st, x, n)
    B.set_option(B.OPT_ROWS_CHUNKS, chunks)
    try:
        for loaded in {8 // chunks, n}:   # one block to a group of wavefronts, and all
            want = ref if loaded == n else O.forward_dense(st, x, loaded)
            for b in (1, 2, 31, 32, 33, 64, 65, 200):
                for dt in (torch.float32, torch.float16):
                    y = torch.full((b, out), float("nan"), dtype=dt, device="cuda:0")
                    ps.linear_batched(torch.from_numpy(x[:b]).to("cuda:0"), loaded, y, kernel=B.KERNEL_PANEL)
                    torch.cuda.synchronize()
                    err = O.relative_error(y.float().cpu().numpy(), want[:b])
                    assert err <= 2e-3, (loaded, b, dt, err)   # also false for an element that was not written (NaN)
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)


@pytest.mark.parametrize("chunks,out,inn,n", shares([(32, 256, 8), (96, 512, 2), (160, 768, 3), (64, 1280, 5), (352, 2304, 9)]))
@pytest.mark.parametrize("batch", [2, 31, 33, 64, 65, 200])
def test_whole_numbers_of_every_share(chunks, out, inn, n, batch):
    import paper_2410_23918_amd as B
    ps, w = stack(out, inn, n, 200)
    x = activations(batch, inn, batch)
    B.set_option(B.OPT_ROWS_CHUNKS, chunks)
    try:
        compare(ps, w, n, x, lambda y: ps.linear_batched(x, n, y, kernel=B.KERNEL_PANEL))
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)


@pytest.mark.parametrize("chunks", [1, 2, 4, 8])
@pytest.mark.parametrize("batch", [2, 32, 40, 130])   # one group of 32 tokens to a workgroup, and two
def test_whole_numbers_over_scales_out_of_fp16_range(chunks, batch):
    """W'/s beyond fp16's largest value in three channels: the workgroup starts over with 1/s on the activations."""
    import paper_2410_23918_amd as B
    small = (5, 300, 767)
    ps, w = stack(96, 768, 11, 130, small)
    x = activations(batch, 768, batch, small)
    B.set_option(B.OPT_ROWS_CHUNKS, chunks)
    try:
        compare(ps, w, 11, x, lambda y: ps.linear_batched(x, 11, y, kernel=B.KERNEL_PANEL))
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)


@pytest.mark.parametrize("chunks", [1, 2, 4])
def test_shares_differ_by_the_order_of_the_sums(chunks):
    """The blocks' sums meet in fp32 before the weight is rounded: another order moves an element by some 2^-24 of the blocks' absolute sum,
    which turns one rounding to fp16 (2^-11) in about a thousand: sqrt(1e-3) 2^-12 = 8e-6 of y in the root mean square.  That they differ at all
shows that the share asked for is the one that ran, and that it was not another kernel."""
    import torch
    import paper_2410_23918_amd as B
    out, inn, n = 320, 1024, 12
    st = synth_stack(2, out, inn, n, tag=5)
    ps = B.PackedStack(st.sign_words(), st.U, st.V, st.s, max_batch=64)
    x = torch.from_numpy(acts(2, 48, inn, tag=5)).to("cuda:0")
    y = {}
    try:
        for c in (chunks, 8, 16):   # 16: without k_rows
            B.set_option(B.OPT_ROWS_CHUNKS, c)
            y[c] = ps.linear_batched(x, n, out_dtype=torch.float32, kernel=B.KERNEL_PANEL).double()
            torch.cuda.synchronize()
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)
    assert 0.0 < ((y[chunks] - y[8]).norm() / y[8].norm()).item() < 2e-5
    assert not (y[16] == y[chunks]).all() and not (y[16] == y[8]).all()


@pytest.mark.parametrize("chunks", [1, 2, 4, 8])
def test_a_weight_beyond_fp16_over_its_scale(chunks):
    """A channel scaled far down, its activations zero: W'/s is no fp16 number, the sums come out right all the same."""
    import torch
    import paper_2410_23918_amd as B
    out, inn, n = 64, 512, 8
    st = synth_stack(3, out, inn, n, tag=9)
    s = np.array(st.s, dtype=np.float32)
    s[3] = s[300] = 1e-8
    x = acts(3, 40, inn, tag=9)
    x[:, [3, 300]] = 0
    ps = B.PackedStack(st.sign_words(), st.U, st.V, s, max_batch=64)
    want = O.forward_dense(O.Stack(st.S, st.U, st.V, s), x, n)
    B.set_option(B.OPT_ROWS_CHUNKS, chunks)
    try:
        y = ps.linear_batched(torch.from_numpy(x).to("cuda:0"), n, kernel=B.KERNEL_PANEL)
        torch.cuda.synchronize()
    finally:
        B.set_option(B.OPT_ROWS_CHUNKS, 0)
    assert O.relative_error(y.float().cpu().numpy(), want) <= 2e-3
