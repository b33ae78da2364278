"""Parity of the HIP path (through the C ABI) with the CPU oracle on the same seeded
inputs.  Tolerance: max_o |y - y_ref| / max_o |y_ref| <= 2e-3 per token (fp16 in,
fp32 accumulate, fp16 out); sign packing and the device-layout round trip bit-exact."""
import ctypes as C

import numpy as np
import pytest

from oracle import bitstack_oracle as O
from workloads import synth as W

from _cases import acts, synth_stack, true_stack

pytestmark = pytest.mark.gpu
TOL = 2e-3


@pytest.fixture(scope="module")
def B():
    import torch
    assert torch.cuda.is_available(), "GPU tests need a GPU"
    import paper_2410_23918_amd as B
    B.lib()
    return B


def _to_dev(x):
    import torch
    return torch.from_numpy(np.ascontiguousarray(x)).to("cuda:0")


def _run(B, ps, x, n_loaded, kernel, dtype="f16"):
    import torch
    xd = _to_dev(x)
    dt = torch.float16 if dtype == "f16" else torch.float32
    y = ps.linear_batched(xd, n_loaded, out_dtype=dt, kernel=kernel)
    torch.cuda.synchronize()
    return y.float().cpu().numpy().astype(np.float64)


def _report(tag, y, ref):
    """The asserted figure (per-row max error over the row's peak) with its two companions."""
    err = O.relative_error(y, ref)
    print(f"{tag}: rel err {err:.2e} (rms-relative {O.rms_relative_error(y, ref):.2e}, "
          f"damped element-wise {O.damped_elementwise_error(y, ref):.2e})", flush=True)
    return err


def _pack(B, st, max_batch=1):
    return B.PackedStack(st.sign_words(), st.U, st.V, st.s, max_batch=max_batch)


# ------------------------------------------------------------------ config 1
def test_cfg1_all_prefixes_both_kernels(B):
    st = true_stack(1, 512, 512, 4)
    ps = _pack(B, st)
    x = acts(1, 1, 512)
    for nl in range(5):
        ref = O.forward_dense(st, x, nl)
        for kern in (B.KERNEL_REFERENCE, B.KERNEL_DECODE):
            for dt in ("f16", "f32"):
                y = _run(B, ps, x, nl, kern, dt)
                if nl == 0:
                    assert not y.any()
                else:
                    err = O.relative_error(y, ref)
                    print(f"cfg1 n_loaded={nl} kernel={kern} {dt}: rel err {err:.2e}", flush=True)
                    assert err <= TOL
    # dense and factored oracle forms agree on the same inputs (config 1's own check)
    assert O.relative_error(O.forward_factored(st, x, 4), O.forward_dense(st, x, 4)) < 1e-12


def test_cfg1_packing_is_bit_exact(B):
    st = true_stack(1, 512, 512, 4)
    # library's canonical sign packing of the float residuals == oracle's
    rng = W.rng_for(1, 0)
    Wt = W.dense_weight(rng, 512, 512, 0.02, False)
    s = W.column_scales(rng, 512)
    R = Wt.astype(np.float64) * s[None, :]
    sw = st.sign_words()
    for i in range(4):
        assert np.array_equal(B.pack_signs_from_f32(R.astype(np.float32)), O.pack_signs(O.sign_pm1(R.astype(np.float32))))
        assert np.array_equal(O.pack_signs(O.sign_pm1(R)), sw[i])
        R = R - O.block_dense(st.S[i], st.U[i], st.V[i])
    ps = _pack(B, st)
    for i in range(4):
        sw2, U2, V2 = ps.unpack_block(i)
        assert np.array_equal(sw2, sw[i])
        assert np.array_equal(U2.view(np.uint16), st.U[i].view(np.uint16))
        assert np.array_equal(V2.view(np.uint16), st.V[i].view(np.uint16))


def test_repeat_calls_leave_workspace_clean(B):
    st = true_stack(1, 512, 512, 4)
    ps = _pack(B, st)
    x = acts(1, 1, 512)
    ref = O.forward_dense(st, x, 4)
    for it in range(5):
        nl = [4, 2, 4, 0, 4][it]
        y = _run(B, ps, x, nl, B.KERNEL_DECODE)
        want = O.forward_dense(st, x, nl)
        if nl:
            assert O.relative_error(y, want) <= TOL
        else:
            assert not y.any()


# ------------------------------------------------------------------ edge shapes
@pytest.mark.parametrize("out,inn,n", [(32, 256, 1), (96, 768, 3), (160, 1024, 2), (1056, 512, 2),
                                       (192, 1536, 2), (64, 2048, 5), (2080, 2048, 3)])
def test_small_and_ragged_shapes(B, out, inn, n):
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=3)
    x = acts(3, 3, inn)
    ref = O.forward_dense(st, x, n)
    y = _run(B, ps, x, n, B.KERNEL_REFERENCE)
    assert O.relative_error(y, ref) <= TOL
    for dt in ("f16", "f32"):
        y = _run(B, ps, x, n, B.KERNEL_PANEL, dt)
        err = O.relative_error(y, ref)
        print(f"{out}x{inn} panel kernel B=3 {dt}: {err:.2e}", flush=True)
        assert err <= TOL
    # forced work splits of the decode kernel: rows per workgroup (tiles per wavefront), chunks per
    # column range (ragged last ranges and last intervals included), block groups, early window
    chunks = inn // 256
    for tiles in (2, 4):
        for ksc in sorted({1, 3, 4, 8, chunks} & set(range(1, min(chunks, 32) + 1))):
            for bg in (0, 1, n):
                for early in ((0, 1, 2, 4) if bg == 0 and ksc in (4, chunks) else (2,)):
                    B.set_option(B.OPT_DECODE_TILES, tiles)
                    B.set_option(B.OPT_DECODE_KS_CHUNKS, ksc)
                    B.set_option(B.OPT_DECODE_BGROUPS, bg)
                    B.set_option(B.OPT_DECODE_EARLY, early + 1)
                    try:
                        y1 = _run(B, ps, x[:1], n, B.KERNEL_DECODE)
                    except B.BitStackError:
                        y1 = None   # the stack's workspace has no room for this split: refused before any launch
                    finally:
                        for opt in (B.OPT_DECODE_TILES, B.OPT_DECODE_KS_CHUNKS, B.OPT_DECODE_BGROUPS, B.OPT_DECODE_EARLY):
                            B.set_option(opt, 0)
                    if y1 is None:
                        assert ksc < 4   # only ranges narrower than the workspace was sized for
                        continue
                    err = O.relative_error(y1, ref[:1])
                    print(f"{out}x{inn} tiles={tiles} ks_chunks={ksc} bgroups={bg} early={early}: {err:.2e}", flush=True)
                    assert err <= TOL


@pytest.mark.parametrize("out,inn,n", [(1056, 768, 3), (96, 2048, 2)])
def test_batch_kernels_every_tile_variant(B, out, inn, n):
    """Batch sizes on both sides of every switch inside the batch path: one / two token groups
    of the small-batch kernel, one / two / four token tiles of the weight-tile kernel, each with
    a ragged last group, an odd number of column chunks and an odd number of row tiles."""
    st = synth_stack(3, out, inn, n)
    batches = (1, 31, 32, 33, 64, 65, 128, 129, 257, 300, 513)
    ps = _pack(B, st, max_batch=max(batches))
    x = acts(3, max(batches), inn)
    ref = O.forward_dense(st, x, n)
    for b in batches:
        for nl in (1, n):
            want = ref[:b] if nl == n else O.forward_dense(st, x[:b], nl)
            y = _run(B, ps, x[:b], nl, B.KERNEL_PANEL)
            assert y.shape == (b, out)
            err = O.relative_error(y, want)
            print(f"{out}x{inn} batch kernel B={b} n_loaded={nl}: {err:.2e}", flush=True)
            assert err <= TOL


def test_batch_kernels_tall_stacks_fall_back(B):
    """Stacks taller than the LDS cache of U rows in the two main batch kernels allows (44 and
    29 blocks) are served by the weight-tile kernel that reads U from memory."""
    out, inn, n = 64, 512, 46
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=200)
    x = acts(3, 200, inn)
    for b, nl in ((2, 46), (2, 44), (70, 46), (70, 30), (70, 29), (200, 31)):
        want = O.forward_dense(st, x[:b], nl)
        y = _run(B, ps, x[:b], nl, B.KERNEL_PANEL)
        err = O.relative_error(y, want)
        print(f"{out}x{inn} batch kernel B={b} n_loaded={nl}: {err:.2e}", flush=True)
        assert err <= TOL


def test_small_batch_column_split_repeatable(B):
    """Few row tiles: the small-batch kernel splits the columns over several workgroups whose
    partial tiles meet in the workspace.  Results must not depend on arrival order (bit-identical
    repeats), the counters must be left at zero (a decode call and another batch call follow), and
    an odd split of the chunks (7 chunks over 3 ranges) must cover every column once."""
    for out, inn, n, b in ((64, 4096, 6, 5), (160, 1792, 8, 2), (4096, 4096, 4, 16)):
        st = synth_stack(3, out, inn, n)
        ps = _pack(B, st, max_batch=b)
        x = acts(3, b, inn)
        ref = O.forward_dense(st, x, n)
        first = None
        for rep in range(3):
            y = _run(B, ps, x, n, B.KERNEL_PANEL, "f32")
            err = O.relative_error(y, ref)
            assert err <= TOL, (out, inn, b, err)
            if first is None:
                first = y
            else:
                assert np.array_equal(first, y)
            y1 = _run(B, ps, x[:1], n, B.KERNEL_DECODE)
            assert O.relative_error(y1, ref[:1]) <= TOL
        print(f"{out}x{inn} n={n} B={b} column split: {err:.2e}", flush=True)
        del ps


def test_blocks_loaded_and_offloaded_one_at_a_time(B):
    """Section 2.2's use case: a stack grows and shrinks block by block.  After every push the
    forward pass over the resident prefix matches the oracle; a popped slot can be refilled with a
    different block; asking for more blocks than are resident is an error; byte accounting follows
    Eq. 9."""
    import torch
    out, inn, n = 1056, 1024, 5
    st = synth_stack(3, out, inn, n)
    other = synth_stack(3, out, inn, n, tag=9)
    sw, sw_o = st.sign_words(), other.sign_words()
    ps = B.PackedStack.empty(out, inn, 4, st.s, max_batch=3)
    assert ps.resident_blocks == 0 and ps.resident_bytes == 0
    x = acts(3, 3, inn)
    y0 = _run(B, ps, x[:1], 0, B.KERNEL_AUTO)
    assert not y0.any()
    for i in range(4):
        ps.push_block(sw[i], st.U[i], st.V[i])
        assert ps.resident_blocks == i + 1 and ps.resident_bytes == (i + 1) * B.block_bytes(out, inn)
        for b, kern in ((1, B.KERNEL_DECODE), (3, B.KERNEL_PANEL)):
            y = _run(B, ps, x[:b], i + 1, kern)
            err = O.relative_error(y, O.forward_dense(st, x[:b], i + 1))
            print(f"push {i}: B={b} rel err {err:.2e}", flush=True)
            assert err <= TOL
    with pytest.raises(B.BitStackError):          # every slot is taken
        ps.push_block(sw[4], st.U[4], st.V[4])
    torch.cuda.synchronize()
    ps.pop_block()
    ps.pop_block()
    assert ps.resident_blocks == 2
    with pytest.raises(B.BitStackError):          # block 2 is not resident any more
        ps.linear(_to_dev(x[0]), 3)
    # refill the freed slots with blocks of another decomposition: a mixed stack
    ps.push_block(sw_o[2], other.U[2], other.V[2])
    ps.push_block(sw_o[3], other.U[3], other.V[3])
    mixed = O.Stack(np.concatenate([st.S[:2], other.S[2:4]]), np.concatenate([st.U[:2], other.U[2:4]]),
                    np.concatenate([st.V[:2], other.V[2:4]]), st.s)
    y = _run(B, ps, x[:1], 4, B.KERNEL_DECODE)
    assert O.relative_error(y, O.forward_dense(mixed, x[:1], 4)) <= TOL
    sw2, U2, V2 = ps.unpack_block(3)
    assert np.array_equal(sw2, sw_o[3]) and np.array_equal(U2.view(np.uint16), other.U[3].view(np.uint16))
    while ps.resident_blocks:
        ps.pop_block()
    with pytest.raises(B.BitStackError):
        ps.pop_block()


def test_job_list_merging_rules(B):
    """Jobs that read one x are merged four at a time; a stack that appears twice, an output that
    overlaps x or another output, or a different input width end a group.  Whatever the grouping,
    every job's output must equal that of its own single launch (all of these take the same kernel
    with one partial row order either way; stacks of mixed sizes: tests/test_gpu_token.py)."""
    import torch
    stacks = [_pack(B, synth_stack(3, 160, 1024, 3, tag=t)) for t in range(6)]
    wide = _pack(B, synth_stack(3, 96, 2048, 2, tag=7))
    x = _to_dev(acts(3, 1, 1024)[0])
    xw = _to_dev(acts(3, 1, 2048)[0])
    big = torch.zeros(1024 + 160, dtype=torch.float16, device="cuda:0")
    big[:1024] = x
    ys = [torch.full((160,), float("nan"), dtype=torch.float16, device="cuda:0") for _ in range(9)]
    yw = torch.full((96,), float("nan"), dtype=torch.float16, device="cuda:0")
    items = [
        (x, stacks[0], 3, ys[0]), (x, stacks[1], 2, ys[1]), (x, stacks[2], 3, ys[2]), (x, stacks[3], 1, ys[3]),
        (x, stacks[4], 3, ys[4]),                      # fifth of a run: starts a new group
        (x, stacks[4], 2, ys[5]),                      # same stack again: its workspace is taken
        (x, stacks[5], 0, ys[6]),                      # empty prefix: y = 0, never merged
        (xw, wide, 2, yw),                             # other input
        (big[:1024], stacks[0], 3, big[1024:]),        # output right behind its input in one buffer: fine
        (x, stacks[1], 3, ys[7]), (x, stacks[2], 3, ys[7]),   # two jobs writing one output: not merged, last wins
    ]
    B.linear_many(B.make_jobs(items))
    torch.cuda.synchronize()
    got = [it[3].clone() for it in items]
    for k, (xi, ps, nl, y) in enumerate(items):
        want = ps.linear(xi, nl)
        torch.cuda.synchronize()
        if k == 9:
            continue                                   # overwritten by job 10
        assert torch.equal(got[k], want), k


@pytest.mark.parametrize("out,inn,n_slots", [(1056, 2048, 6), (4096, 4096, 16), (2048, 1024, 2)])
def test_small_batch_through_the_decode_kernel(B, out, inn, n_slots):
    """Batches of 2..9 tokens through the decode kernel: up to four tokens share a launch, each
    with its own activation row, output row and piece of the stack's split-accumulation workspace
    (the third shape has a workspace too small for four, so the launcher falls back to fewer per
    launch).  Every token against the oracle; a second pass over the same buffers checks that the
    arrival counters were left at zero; the single-token result is unchanged afterwards."""
    st = synth_stack(3, out, inn, n_slots, tag=9)
    ps = _pack(B, st, max_batch=16)
    x = acts(3, 9, inn, tag=9)
    for nl in sorted({1, n_slots // 2, n_slots} - {0}):
        ref = O.forward_dense(st, x, nl)
        for b in (2, 3, 4, 5, 9):
            for rep in range(2):
                y = _run(B, ps, x[:b], nl, B.KERNEL_DECODE, "f32" if rep else "f16")
                assert y.shape == (b, out)
                err = O.relative_error(y, ref[:b])
                print(f"{out}x{inn} n_loaded={nl} B={b} pass {rep}: {err:.2e}", flush=True)
                assert err <= TOL
        y1 = _run(B, ps, x[:1], nl, B.KERNEL_DECODE)
        assert O.relative_error(y1, ref[:1]) <= TOL


@pytest.mark.parametrize("tiles", [0, 2, 4])
def test_degenerate_activations(B, tiles):
    """x = 0 gives y = 0 exactly (the panel's quantisation scale is zero: nothing may divide by
    it); a one-hot x picks one column of W' diag(1/s); a huge and a tiny x keep the relative error
    (the panel is quantised against its own maximum per block and column slab).  One token through this
    stack is k_token's; a forced work split sends it to k_decode."""
    B.set_option(B.OPT_DECODE_TILES, tiles)
    try:
        degenerate_activations(B)
    finally:
        B.set_option(B.OPT_DECODE_TILES, 0)


def degenerate_activations(B):
    import torch
    out, inn, n = 1056, 2048, 3
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=40)
    zero = np.zeros((1, inn), dtype=np.float16)
    for kern in (B.KERNEL_DECODE, B.KERNEL_PANEL, B.KERNEL_REFERENCE):
        y = _run(B, ps, zero, n, kern)
        assert not y.any() and np.isfinite(y).all()
    hot = np.zeros((3, inn), dtype=np.float16)
    hot[0, 0] = 1.0
    hot[1, 1023] = -2.5
    hot[2, inn - 1] = 0.125
    ref = O.forward_dense(st, hot, n)
    for kern in (B.KERNEL_DECODE, B.KERNEL_PANEL):
        y = _run(B, ps, hot, n, kern)
        err = O.relative_error(y, ref)
        print(f"one-hot activations, kernel {kern}: {err:.2e}", flush=True)
        assert err <= TOL
    x = acts(3, 1, inn)
    for scale in (2.0 ** -14, 2.0 ** 10):
        xs = (x.astype(np.float32) * scale).astype(np.float16)
        want = O.forward_dense(st, xs, n)
        if np.abs(want).max() < 6.0e4:                      # stays inside fp16's range
            y = _run(B, ps, xs, n, B.KERNEL_DECODE)
            err = O.relative_error(y, want)
            print(f"activations scaled by {scale:g}: {err:.2e}", flush=True)
            assert err <= TOL
        y32 = _run(B, ps, xs, n, B.KERNEL_DECODE, "f32")
        assert O.relative_error(y32, want) <= TOL


def _outlier_activations(inn):
    """x ~ N(0,1) with 1, 4 and 32 channels at 30x and 100x, 1 and 4 at 1000x, and a Student-t(3)
    draw: a few channels far above the rest is the situation activation-aware scaling (Eq. 3-4)
    exists for."""
    base = acts(2, 1, inn, tag=9).astype(np.float32)
    cases = []
    for fac, counts in ((30.0, (1, 4, 32)), (100.0, (1, 4, 32)), (1000.0, (1, 4))):
        for cnt in counts:
            x = base.copy()
            x[0, W.rng_for(2, 77, cnt, int(fac)).choice(inn, cnt, replace=False)] *= fac
            cases.append((f"{cnt} channel(s) x{fac:g}", x.astype(np.float16)))
    t3 = W.rng_for(2, 78, inn).standard_t(3, size=(1, inn)).astype(np.float32)
    cases.append(("Student-t(3)", t3.astype(np.float16)))
    return cases


@pytest.mark.parametrize("out,inn,n,true_iavd", [(4096, 4096, 16, True), (1056, 2048, 5, False)])
def test_outlier_activations(B, out, inn, n, true_iavd):
    st = true_stack(2, out, inn, n, method="subspace", iters=30) if true_iavd else synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=2)
    chunks = inn // 256
    for tag, x in _outlier_activations(inn):
        ref = O.forward_dense(st, x, n)
        # decode kernel: its own choice of work split, one range over the whole row, ranges of one interval
        for tiles, ksc in ((0, 0), (4, min(chunks, 32)), (2, 4)):
            B.set_option(B.OPT_DECODE_TILES, tiles)
            B.set_option(B.OPT_DECODE_KS_CHUNKS, ksc)
            try:
                y = _run(B, ps, x, n, B.KERNEL_DECODE)
            finally:
                B.set_option(B.OPT_DECODE_TILES, 0)
                B.set_option(B.OPT_DECODE_KS_CHUNKS, 0)
            err = _report(f"{out}x{inn} {tag}, decode kernel tiles={tiles} ks_chunks={ksc}", y, ref)
            assert err <= TOL
        y = _run(B, ps, x, n, B.KERNEL_PANEL)
        err = _report(f"{out}x{inn} {tag}, batch kernel", y, ref)
        assert err <= TOL


def test_mlp_shaped_true_decomposition(B):
    """A 14336x4096 stack from the oracle's own decomposition (subspace iteration run to
    convergence, 4 blocks) through the decode kernel and the batch kernels."""
    st = true_stack(3, 14336, 4096, 4, method="subspace", iters=30)
    ps = _pack(B, st, max_batch=16)
    x = acts(3, 16, 4096, tag=5)
    ref = O.forward_dense(st, x, 4)
    for b, kern, name in ((1, B.KERNEL_DECODE, "decode"), (3, B.KERNEL_DECODE, "decode"), (16, B.KERNEL_PANEL, "batch"),
                          (16, B.KERNEL_AUTO, "library's choice")):
        y = _run(B, ps, x[:b], 4, kern)
        err = _report(f"14336x4096 true decomposition n=4, {b} token(s), {name} kernel", y, ref[:b])
        assert err <= TOL


def test_two_stacks_on_two_streams(B):
    """Calls on different handles may overlap in time (each image has its own workspace and
    counters; the library keeps no per-call state of its own): two stacks driven from two streams
    give the same bits as one after the other."""
    import torch
    a = synth_stack(3, 1056, 2048, 3)
    b = synth_stack(3, 2048, 1024, 4, tag=1)
    pa, pb = _pack(B, a), _pack(B, b)
    xa = torch.from_numpy(acts(3, 1, 2048)[0]).to("cuda:0")
    xb = torch.from_numpy(acts(3, 1, 1024, tag=1)[0]).to("cuda:0")
    ya_ref = pa.linear(xa, 3).clone()
    yb_ref = pb.linear(xb, 4).clone()
    torch.cuda.synchronize()
    s1, s2 = torch.cuda.Stream(), torch.cuda.Stream()      # default priority
    ya = [torch.empty_like(ya_ref) for _ in range(20)]
    yb = [torch.empty_like(yb_ref) for _ in range(20)]
    for i in range(20):
        pa.linear(xa, 3, y=ya[i], stream=s1)
        pb.linear(xb, 4, y=yb[i], stream=s2)
    s1.synchronize()
    s2.synchronize()
    for i in range(20):
        assert torch.equal(ya[i], ya_ref) and torch.equal(yb[i], yb_ref)
    err = O.relative_error(ya_ref.float().cpu().numpy()[None], O.forward_dense(a, acts(3, 1, 2048), 3))
    assert err <= TOL


def test_argument_errors_on_device(B):
    import torch
    st = synth_stack(3, 32, 256, 1)
    ps = _pack(B, st, max_batch=2)
    L = B.lib()
    x = torch.zeros(2 * 256 + 8, dtype=torch.float16, device="cuda:0")
    y = torch.zeros(2 * 32 + 8, dtype=torch.float16, device="cuda:0")
    s0 = C.c_void_p(0)
    assert L.bitstack_linear(x.data_ptr(), ps.handle, 2, y.data_ptr(), s0) == -3      # n_loaded > n
    assert L.bitstack_linear(x.data_ptr(), ps.handle, -1, y.data_ptr(), s0) == -3
    assert L.bitstack_linear(x.data_ptr() + 2, ps.handle, 1, y.data_ptr(), s0) == -4  # misaligned
    assert L.bitstack_linear_batched(x.data_ptr(), 3, ps.handle, 1, y.data_ptr(), 0, s0) == -3  # batch > max
    assert L.bitstack_linear_batched(x.data_ptr(), 1, ps.handle, 1, y.data_ptr(), 7, s0) == -8
    assert L.bitstack_linear_select(x.data_ptr(), 1, ps.handle, 1, y.data_ptr(), 0, 9, s0) == -8
    assert L.bitstack_unpack_blocks(ps.handle, 5, None, None, None, s0) == -3
    torch.cuda.synchronize()


# ------------------------------------------------------------------ config 2
def test_cfg2_llama_attn_proj_true_iavd(B):
    # subspace iteration with 32 columns run to convergence (30 rounds): a true decomposition
    st = true_stack(2, 4096, 4096, 16, method="subspace", iters=30)
    ps = _pack(B, st)
    x = acts(2, 1, 4096)
    for nl in (16, 7, 1):
        ref = O.forward_dense(st, x, nl)
        for kern in (B.KERNEL_DECODE, B.KERNEL_REFERENCE):
            y = _run(B, ps, x, nl, kern)
            err = _report(f"cfg2 n_loaded={nl} kernel={kern}", y, ref)
            assert err <= TOL
    # few block groups: a workgroup walks through many blocks (more than the number whose slab
    # maxima are prepared before the first barrier), many partial rows per row slab otherwise
    ref = O.forward_dense(st, x, 16)
    for bg in (1, 2, 3, 16):
        B.set_option(B.OPT_DECODE_BGROUPS, bg)
        try:
            y = _run(B, ps, x, 16, B.KERNEL_DECODE)
        finally:
            B.set_option(B.OPT_DECODE_BGROUPS, 0)
        err = O.relative_error(y, ref)
        print(f"cfg2 n_loaded=16 block groups={bg}: rel err {err:.2e}", flush=True)
        assert err <= TOL
    sw2, U2, V2 = ps.unpack_block(15)
    assert np.array_equal(sw2, st.sign_words()[15])


# ------------------------------------------------------------------ config 3
@pytest.mark.parametrize("out,inn", [(14336, 4096), (4096, 14336)])
def test_cfg3_llama_mlp_batches(B, out, inn):
    st = synth_stack(3, out, inn, 16)
    ps = _pack(B, st, max_batch=16)
    x = acts(3, 16, inn)
    ref = O.forward_dense(st, x, 16)
    y = _run(B, ps, x[:1], 16, B.KERNEL_DECODE)
    err = O.relative_error(y, ref[:1])
    print(f"cfg3 {out}x{inn} B=1 decode: {err:.2e}", flush=True)
    assert err <= TOL
    for b in (1, 4, 16):
        y = _run(B, ps, x[:b], 16, B.KERNEL_AUTO)
        err = O.relative_error(y, ref[:b])
        print(f"cfg3 {out}x{inn} B={b} auto: {err:.2e}", flush=True)
        assert err <= TOL
    for b in (1, 16):
        y = _run(B, ps, x[:b], 16, B.KERNEL_PANEL)
        err = O.relative_error(y, ref[:b])
        print(f"cfg3 {out}x{inn} B={b} panel kernel: {err:.2e}", flush=True)
        assert err <= TOL
    y = _run(B, ps, x[:16], 16, B.KERNEL_REFERENCE, "f32")
    err = O.relative_error(y, ref[:16])
    print(f"cfg3 {out}x{inn} B=16 reference kernel: {err:.2e}", flush=True)
    assert err <= TOL


# ------------------------------------------------------------------ config 4
def test_cfg4_decoder_layer_variable_stack_heights(B):
    rng = W.rng_for(4, 0)
    nl_all = W.variable_n_loaded(rng, 32 * 7)
    assert nl_all.min() >= 8 and nl_all.max() <= 24
    rows_rng = W.rng_for(4, 1)
    for m, (name, out, inn) in enumerate(W.llama3_8b_layer_shapes()):
        draws = (int(nl_all[m]), int(nl_all[7 + m]))   # this matrix in layers 0 and 1
        st = synth_stack(4, out, inn, max(draws), tag=m)   # blocks past n_loaded are never read
        ps = _pack(B, st)
        x = acts(4, 1, inn, tag=m)
        # rows from every 1024-row slab (every row slab of the decode kernel, both tile heights)
        rows = np.sort(np.concatenate([lo + rows_rng.choice(min(1024, out - lo), size=48, replace=False)
                                       for lo in range(0, out, 1024)]))
        for layer, nl in enumerate(draws):
            ref = O.forward_rows(st, x, nl, rows)
            y = _run(B, ps, x, nl, B.KERNEL_AUTO)
            # sampled rows; scale by the max over the sample
            err = _report(f"cfg4 layer {layer} {name} {out}x{inn} n_loaded={nl} ({len(rows)} rows)", y[:, rows], ref)
            assert err <= TOL
        del ps
    synth_stack.cache_clear()


def test_cfg4_layer_through_one_native_call_with_merged_launches(B):
    """The seven linears of a decoder layer as one job list: q/k/v read one vector, gate/up
    another, so the native loop merges them into grouped launches (3 + 1 + 2 + 1 jobs).  Every
    output is checked against the oracle on sampled rows and against its own single launch; a
    second pass over the same list checks that the workspaces were left clean."""
    import torch
    rng = W.rng_for(4, 0)
    nl_all = W.variable_n_loaded(rng, 32 * 7)
    shapes = W.llama3_8b_layer_shapes()
    xs = {4096: _to_dev(acts(4, 1, 4096, tag=100)[0]), 14336: _to_dev(acts(4, 1, 14336, tag=101)[0])}
    x_o = _to_dev(acts(4, 1, 4096, tag=102)[0])
    items, keep = [], []
    for m, (name, out, inn) in enumerate(shapes):
        nl = int(nl_all[m])
        st = synth_stack(4, out, inn, nl, tag=m)
        ps = _pack(B, st)
        x = x_o if name == "o_proj" else xs[inn]
        y = torch.full((out,), float("nan"), dtype=torch.float16, device="cuda:0")
        items.append((x, ps, nl, y))
        keep.append((name, st, nl))
    jobs = B.make_jobs(items)
    rows_rng = W.rng_for(4, 2)
    for rep in range(2):
        for it in items:
            it[3].fill_(float("nan"))
        B.linear_many(jobs)
        torch.cuda.synchronize()
        for (name, st, nl), (x, ps, _, y) in zip(keep, items):
            out = y.shape[0]
            rows = np.sort(rows_rng.choice(out, size=128, replace=False))
            xin = x.cpu().numpy()[None, :]
            ref = O.forward_rows(st, xin, nl, rows)
            got = y.float().cpu().numpy().astype(np.float64)[None, :]
            assert np.isfinite(got).all()
            err = O.relative_error(got[:, rows], ref)
            single = ps.linear(x, nl).float().cpu().numpy().astype(np.float64)[None, :]
            dev = O.relative_error(got, single)
            print(f"cfg4 merged pass {rep} {name} n_loaded={nl}: vs oracle {err:.2e}, vs single launch {dev:.2e}", flush=True)
            assert err <= TOL and dev <= 1e-3
    del jobs, items
    synth_stack.cache_clear()


# ------------------------------------------------------------------ materialising path
@pytest.mark.parametrize("out,inn,n", [(1056, 768, 3), (96, 2048, 2), (64, 512, 29)])
def test_restored_weight_matches_eq8(B, out, inn, n):
    """The dense matrix the restore kernel writes against Eq. 8 with the scaling of Eq. 4 folded
    into the columns, element by element: per output row, max_j |w - w_ref| / max_j |w_ref|
    (the blocks are summed in fp32, the weight is rounded to fp16 once)."""
    import torch
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=65)
    assert B.dense_bytes(out, inn) == out * inn * 2
    guard = 512
    buf = torch.full((out * inn + 2 * guard,), 7.0, dtype=torch.float16, device="cuda:0")
    wd = buf[guard:guard + out * inn].view(out, inn)
    assert wd.data_ptr() % 256 == 0
    for nl in sorted({0, 1, n // 2 + 1, n}):
        ps.restore_weight(nl, wd)
        torch.cuda.synchronize()
        got = wd.float().cpu().numpy().astype(np.float64)
        ref = O.reconstruct_scaled(st, nl) / np.asarray(st.s, dtype=np.float64)[None, :]
        if nl == 0:
            assert not got.any()
        else:
            err = O.relative_error(got, ref)
            print(f"{out}x{inn} restored weight n_loaded={nl}: {err:.2e}", flush=True)
            assert err <= TOL
        assert (buf[:guard] == 7.0).all() and (buf[guard + out * inn:] == 7.0).all()   # nothing written outside
    assert B.restore_max_blocks() == 29


@pytest.mark.parametrize("out,inn,n", [(1056, 768, 3), (96, 2048, 2)])
def test_materialised_path_every_tile_variant(B, out, inn, n):
    """Restore + dense product against the oracle for batches on both sides of the product
    kernel's tiles (32-token fragments, 64 tokens per wavefront, 128 or 256 per workgroup), with
    ragged row tiles (out not a multiple of 128 or 256), both output types and each of the four
    output tiles of the product forced in turn (256 x 256, 128 x 256, 128 x 128 with the columns
    of a chunk split over the two halves of the workgroup, 128 x 128 with the columns split over
    four pairs of wavefronts), then the launcher's own choice; the two-step form (restore once, multiply many times) gives the same bits as the combined call."""
    import torch
    st = synth_stack(3, out, inn, n)
    batches = (1, 31, 33, 64, 65, 255, 256, 257, 513)
    ps = _pack(B, st, max_batch=max(batches))
    x = acts(3, max(batches), inn)
    ref = O.forward_dense(st, x, n)
    wd = torch.empty((out, inn), dtype=torch.float16, device="cuda:0")
    for b in batches:
        xd = _to_dev(x[:b])
        for dt in (torch.float16, torch.float32):
            for tile in (1, 2, 3, 4, 0):
                B.set_option(B.OPT_DENSE_TILE, tile)
                try:
                    y = ps.linear_materialised(xd, n, wd, out_dtype=dt)
                    y2 = ps.linear_dense(xd, wd, out_dtype=dt)
                    torch.cuda.synchronize()
                finally:
                    B.set_option(B.OPT_DENSE_TILE, 0)
                assert y.shape == (b, out)
                err = O.relative_error(y.float().cpu().numpy(), ref[:b])
                print(f"{out}x{inn} materialised B={b} {dt}, product tile {tile or 'chosen'}: {err:.2e}", flush=True)
                assert err <= TOL
                assert torch.equal(y, y2)
    # a shorter prefix through the same scratch
    y = ps.linear_materialised(_to_dev(x[:70]), 1, wd)
    torch.cuda.synchronize()
    err = O.relative_error(y.float().cpu().numpy(), O.forward_dense(st, x[:70], 1))
    assert err <= TOL
    y = ps.linear_materialised(_to_dev(x[:70]), 0, wd)
    torch.cuda.synchronize()
    assert not y.any()


def test_weight_tile_kernel_takes_33_to_64_tokens_when_row_tiles_are_many(B):
    """For 33..64 tokens the batch launcher takes the weight-tile kernel instead of the small-batch
    one when that is estimated cheaper: here 224 row tiles, where the small-batch kernel would need
    448 workgroups and rebuild every signed tile twice.  Every output against the oracle, on both
    sides of the 32-token groups, both output types."""
    import torch
    out, inn, n = 14336, 512, 3
    st = synth_stack(3, out, inn, n, tag=6)
    ps = _pack(B, st, max_batch=128)
    x = acts(3, 64, inn, tag=6)
    ref = O.forward_dense(st, x, n)
    for b in (33, 48, 64):
        assert B.choose_kernel(out, inn, n, 128, b, n, 0) == B.KERNEL_PANEL
        for dt in (torch.float16, torch.float32):
            y = ps.linear_batched(_to_dev(x[:b]), n, out_dtype=dt, kernel=B.KERNEL_PANEL)
            torch.cuda.synchronize()
            err = O.relative_error(y.float().cpu().numpy(), ref[:b])
            print(f"{out}x{inn} B={b} {dt}: {err:.2e}", flush=True)
            assert err <= TOL


def test_dense_product_with_256_row_tiles(B):
    """The small shapes above all run the product kernel's 128-row tiles (fewer than 129 of the
    256-row ones would leave compute units idle).  This shape has 8 x 17 = 136 tiles of 256 rows
    (one round of the chip) against 272 of 128 rows (two rounds), so it takes the 256-row variant:
    every output against the oracle, with a ragged last row tile (160 rows) and a ragged last token
    tile (104 tokens), both output types."""
    import torch
    out, inn, n, T = 1952, 256, 2, 4200
    st = synth_stack(5, out, inn, n)
    ps = _pack(B, st, max_batch=T)
    x = acts(5, T, inn)
    ref = O.forward_dense(st, x, n)
    wd = torch.empty((out, inn), dtype=torch.float16, device="cuda:0")
    xd = _to_dev(x)
    for dt in (torch.float16, torch.float32):
        y = ps.linear_materialised(xd, n, wd, out_dtype=dt)
        torch.cuda.synchronize()
        err = O.relative_error(y.float().cpu().numpy(), ref)
        print(f"{out}x{inn} materialised B={T} {dt}: {err:.2e}", flush=True)
        assert err <= TOL


def test_library_choice_with_an_optional_scratch_buffer(B):
    """bitstack_linear_batched_ws: same results with and without the scratch buffer; the buffer is
    overwritten exactly when the host-side choice says so, left alone otherwise."""
    import torch
    out, inn, n, T = 8192, 1024, 4, 2048
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=T)
    x = acts(3, T, inn)
    ref = O.forward_dense(st, x, n)
    ws = torch.full((out, inn), 3.0, dtype=torch.float16, device="cuda:0")
    for b in (1, 40, 200, 2048):
        choice = B.choose_kernel(out, inn, n, T, b, n, ws.numel() * 2)
        ws.fill_(3.0)
        xd = _to_dev(x[:b])
        y1 = ps.linear_batched_ws(xd, n, ws)
        y0 = ps.linear_batched_ws(xd, n, None)
        torch.cuda.synchronize()
        touched = bool((ws != 3.0).any())
        print(f"{out}x{inn} B={b}: choice {choice}, scratch touched: {touched}", flush=True)
        assert touched == (choice == B.KERNEL_MATERIALISE)
        for y in (y0, y1):
            err = O.relative_error(y.float().cpu().numpy(), ref[:b])
            assert err <= TOL
    assert B.choose_kernel(out, inn, n, T, 2048, n, ws.numel() * 2) == B.KERNEL_MATERIALISE
    assert B.choose_kernel(out, inn, n, T, 1, n, ws.numel() * 2) == B.KERNEL_DECODE
    # too small a buffer is ignored, a misaligned one is an error
    small = torch.empty(1024, dtype=torch.float16, device="cuda:0")
    y = ps.linear_batched_ws(_to_dev(x), n, small)
    torch.cuda.synchronize()
    assert O.relative_error(y.float().cpu().numpy(), ref) <= TOL
    L = B.lib()
    assert L.bitstack_linear_batched_ws(C.c_void_p(y.data_ptr()), 1, ps.handle, n, C.c_void_p(y.data_ptr()), 0,
                                        C.c_void_p(ws.data_ptr() + 16), ws.numel() * 2, None) == -4


def test_materialised_path_through_the_images_own_scratch(B):
    """No scratch lent: an image packed for many tokens carries max_batch x in fp16 of activation
    scratch (the weight-tile kernel's), which the materialising path uses for slabs of the dense
    weight.  Forced through the kernel selector: same bits as through a caller's scratch for the
    whole matrix when the dense product's tile is held fixed, the parity bound with the launcher's
    own choice per slab; the weight-tile kernel, which writes activations there, still works afterwards;
    an image packed for at most 64 tokens has no such scratch and the selector is refused."""
    import torch
    out, inn, n = 2336, 1024, 3       # 1120 tokens of scratch = 1024 rows at a time: slabs of 1024, 1024, 288
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=1100)
    x = acts(3, 1100, inn)
    ref = O.forward_dense(st, x, n)
    full = torch.empty((out, inn), dtype=torch.float16, device="cuda:0")
    for b in (70, 1100):
        xd = _to_dev(x[:b])
        for dt in (torch.float16, torch.float32):
            for tile in (3, 4):
                B.set_option(B.OPT_DENSE_TILE, tile)
                try:
                    y_full = ps.linear_materialised(xd, n, full, out_dtype=dt)
                    y_img = ps.linear_batched(xd, n, out_dtype=dt, kernel=B.KERNEL_MATERIALISE)
                    torch.cuda.synchronize()
                finally:
                    B.set_option(B.OPT_DENSE_TILE, 0)
                assert torch.equal(y_full, y_img), (b, dt, tile)
            y_img = ps.linear_batched(xd, n, out_dtype=dt, kernel=B.KERNEL_MATERIALISE)
            y_tile = ps.linear_batched(xd, n, out_dtype=dt, kernel=B.KERNEL_PANEL)
            torch.cuda.synchronize()
            for name, y in (("materialised through the image's scratch", y_img), ("batch kernel after it", y_tile)):
                err = _report(f"{out}x{inn} B={b} {dt}, {name}", y.float().cpu().numpy(), ref[:b])
                assert err <= TOL
    # a caller's scratch smaller than the image's is left alone
    small = torch.full((1024 * inn,), 7.0, dtype=torch.float16, device="cuda:0")
    assert B.choose_kernel(out, inn, n, 1100, 1100, n, small.numel() * 2) == B.choose_kernel(out, inn, n, 1100, 1100, n, 0)
    few = _pack(B, st, max_batch=64)
    y = torch.empty((8, out), dtype=torch.float16, device="cuda:0")
    L = B.lib()
    assert L.bitstack_linear_select(C.c_void_p(_to_dev(x[:8]).data_ptr()), 8, few.handle, n, C.c_void_p(y.data_ptr()), 0,
                                    B.KERNEL_MATERIALISE, None) == -6


def test_materialised_path_in_row_slabs_through_a_small_scratch(B):
    """A scratch with room for fewer rows than the weight has: the weight is restored and multiplied
    slab by slab through it.  With the dense product's output tile held fixed (each of its four
    tiles in turn: 256 x 256, 128 x 256, 128 x 128 with the columns of a chunk split over two
    halves of the workgroup, 128 x 128 for long rows) the bits are those of a scratch for the whole matrix -- the same
    kernel does the same arithmetic per row -- for a slab count that leaves a short last slab and
    both output types; with the launcher's own choice of tile per slab the result holds the
    parity bound; a scratch below 1024 rows is refused."""
    import torch
    out, inn, n = 2336, 1024, 3       # 2336 = 2 x 1024 + 288: two full slabs and a ragged one
    st = synth_stack(3, out, inn, n)
    ps = _pack(B, st, max_batch=600)
    x = acts(3, 600, inn)
    ref = O.forward_dense(st, x, n)
    full = torch.empty((out, inn), dtype=torch.float16, device="cuda:0")
    for rows in (1024, 1280, 2304):
        slab = torch.full((rows * inn + 100,), 7.0, dtype=torch.float16, device="cuda:0")[: rows * inn + 60]
        for b in (70, 600):
            xd = _to_dev(x[:b])
            for dt in (torch.float16, torch.float32):
                for tile in (1, 2, 3, 4, 0):
                    B.set_option(B.OPT_DENSE_TILE, tile)
                    try:
                        y_full = ps.linear_materialised(xd, n, full, out_dtype=dt)
                        y_slab = ps.linear_materialised(xd, n, slab, out_dtype=dt)
                        torch.cuda.synchronize()
                    finally:
                        B.set_option(B.OPT_DENSE_TILE, 0)
                    if tile:
                        assert torch.equal(y_full, y_slab), (rows, b, dt, tile)
                    err = O.relative_error(y_slab.float().cpu().numpy(), ref[:b])
                    print(f"{out}x{inn} scratch of {rows} rows, B={b} {dt}, product tile {tile or 'chosen per slab'}: "
                          f"{err:.2e}", flush=True)
                    assert err <= TOL
        assert bool((slab[rows * inn:] == 7.0).all())      # nothing written past the rows that fit
    slab = torch.empty((1024 * inn,), dtype=torch.float16, device="cuda:0")
    y0 = ps.linear_materialised(_to_dev(x[:70]), 0, slab)
    torch.cuda.synchronize()
    assert not y0.any()
    # the library's choice takes the slab path for a prefill-sized batch and gives the same result
    assert B.choose_kernel(out, inn, n, 600, 600, n, slab.numel() * 2) in (B.KERNEL_MATERIALISE, B.KERNEL_PANEL)
    y = ps.linear_batched_ws(_to_dev(x), n, slab)
    torch.cuda.synchronize()
    assert O.relative_error(y.float().cpu().numpy(), ref) <= TOL
    tiny = torch.empty((1023 * inn,), dtype=torch.float16, device="cuda:0")
    with pytest.raises(B.BitStackError) as e:
        ps.linear_materialised(_to_dev(x[:70]), n, tiny)
    assert e.value.code == -6


def test_materialised_path_argument_errors(B):
    import torch
    L = B.lib()
    st = synth_stack(3, 64, 512, 30)
    ps = _pack(B, st, max_batch=100)
    small = _pack(B, st, max_batch=8)
    x = _to_dev(acts(3, 100, 512))
    y = torch.empty((100, 64), dtype=torch.float16, device="cuda:0")
    wd = torch.empty((64 * 512 + 64,), dtype=torch.float16, device="cuda:0")
    nb = 64 * 512 * 2
    vp = C.c_void_p
    assert L.bitstack_restore_weight(ps.handle, 30, vp(wd.data_ptr()), nb, None) == -3      # taller than the U cache
    assert L.bitstack_restore_weight(ps.handle, 31, vp(wd.data_ptr()), nb, None) == -3
    assert L.bitstack_restore_weight(ps.handle, 2, vp(wd.data_ptr()), nb - 2, None) == -6
    assert L.bitstack_restore_weight(ps.handle, 2, vp(wd.data_ptr() + 16), nb, None) == -4
    assert L.bitstack_restore_weight(ps.handle, 2, None, nb, None) == -1
    assert L.bitstack_linear_dense(vp(x.data_ptr()), 101, ps.handle, vp(wd.data_ptr()), vp(y.data_ptr()), 0, None) == -3
    assert L.bitstack_linear_dense(vp(x.data_ptr()), 9, small.handle, vp(wd.data_ptr()), vp(y.data_ptr()), 0, None) == -3
    assert L.bitstack_linear_dense(vp(x.data_ptr()), 8, ps.handle, vp(wd.data_ptr()), vp(y.data_ptr()), 5, None) == -8
    assert L.bitstack_linear_materialised(vp(x.data_ptr()), 8, ps.handle, 2, vp(wd.data_ptr()), nb - 2,
                                          vp(y.data_ptr()), 0, None) == -6
    assert L.bitstack_linear_materialised(vp(x.data_ptr()), 8, ps.handle, 2, vp(wd.data_ptr()), nb,
                                          vp(y.data_ptr()), 0, None) == 0
    torch.cuda.synchronize()
    err = O.relative_error(y[:8].float().cpu().numpy(), O.forward_dense(st, acts(3, 100, 512)[:8], 2))
    assert err <= TOL


# ------------------------------------------------------------------ config 5
def test_cfg5_llama70b_mlp_prefill_sampled(B):
    """28672x8192, n=16, 2048 tokens.  The oracle cannot finish the full product in
    seconds, so one output row of every 64-row tile is compared for every token, the two
    device paths are compared with each other on every output, and the rest is checked
    through properties that hold at any size."""
    import torch
    out, inn, n, T = 28672, 8192, 16, 2048
    st = synth_stack(5, out, inn, n)
    ps = _pack(B, st, max_batch=T)
    x = acts(5, T, inn)
    xd = _to_dev(x)
    y = ps.linear_batched(xd, n)           # fp16 [T, out]
    torch.cuda.synchronize()
    rng = W.rng_for(5, 2)
    # one row of every 64-row workgroup tile (448 rows), every token: each workgroup of the
    # weight-tile kernel and each tile of the dense product contributes to what is compared
    rows = np.arange(0, out, 64) + rng.integers(0, 64, size=out // 64)
    ref = O.forward_rows(st, x, n, rows)                       # (T, 448) in fp64
    rows_d = torch.from_numpy(rows).to("cuda:0")
    got = y[:, rows_d].float().cpu().numpy()
    err = _report(f"cfg5 weight-tile kernel, {T} tokens x {len(rows)} rows (one per 64-row tile)", got, ref)
    assert err <= TOL
    # every output finite, no token left unwritten, and linearity in x on the device path:
    # y(x_a) + y(x_b) vs y(x_a + x_b) for one token (inputs chosen so the sum is exact in fp16)
    assert torch.isfinite(y).all()
    assert (y.abs().amax(dim=1) > 0).all()
    xa = (np.round(x[5].astype(np.float32) * 8) / 8).astype(np.float16)
    xb = (np.round(x[6].astype(np.float32) * 8) / 8).astype(np.float16)
    trio = np.stack([xa, xb, (xa.astype(np.float32) + xb.astype(np.float32)).astype(np.float16)])
    y3 = ps.linear_batched(_to_dev(trio), n, out_dtype=torch.float32).cpu().numpy().astype(np.float64)
    lin = np.abs(y3[0] + y3[1] - y3[2]).max() / np.abs(y3[2]).max()
    print(f"cfg5 linearity residual: {lin:.2e}", flush=True)
    assert lin <= 2 * TOL
    # the materialising path on the same samples
    wd = torch.empty((out, inn), dtype=torch.float16, device="cuda:0")
    ym = ps.linear_materialised(xd, n, wd)
    torch.cuda.synchronize()
    gotm = ym[:, rows_d].float().cpu().numpy()
    errm = _report("cfg5 materialised path, same samples", gotm, ref)
    assert errm <= TOL
    # the two device paths against each other over all 58.7 M outputs (they multiply the same fp16
    # weight tiles; a tile either of them got wrong shows up here whether or not it was sampled)
    worst = 0.0
    for t0 in range(0, T, 256):
        a, b = y[t0:t0 + 256].float(), ym[t0:t0 + 256].float()
        worst = max(worst, ((a - b).abs().amax(dim=1) / b.abs().amax(dim=1)).max().item())
    print(f"cfg5 weight-tile kernel vs materialised path, every output: {worst:.2e}", flush=True)
    assert worst <= TOL
    assert torch.isfinite(ym).all() and (ym.abs().amax(dim=1) > 0).all()
    wrows = wd[rows_d].float().cpu().numpy().astype(np.float64)
    wref = np.zeros((len(rows), inn))
    for i in range(n):
        wref += st.S[i][rows].astype(np.float64) * (st.U[i][rows].astype(np.float64) @ st.V[i].astype(np.float64).T)
    wref /= np.asarray(st.s, dtype=np.float64)[None, :]
    errw = O.relative_error(wrows, wref)
    print(f"cfg5 restored weight, {len(rows)} sampled rows: {errw:.2e}", flush=True)
    assert errw <= TOL
    synth_stack.cache_clear()
