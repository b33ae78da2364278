"""The work that a user of this library has it do, as cases to be timed and compared.

A case is a linear layer held as a stack of residual blocks (out x in, n loaded blocks, rank 16) and one pass through a public
entry point: one token (decode), a decoder layer's seven linears for one token, a batch of tokens (a few sequences decoded
together, a chunk of a prompt, a whole prompt), or the compression of a weight.  Shapes are those of workloads/synth.py, the
benchmark and the tests, stack heights those of the benchmark (8 to 24) and of memory budgets where 2 to 4 blocks are loaded.
"""
import math

import numpy as np
import torch

import paper_2410_23918_amd as B

K = 16
DEV = "cuda:0"
# the linears of a decoder layer that read one vector, in the order a token passes them: (out, in); sizes of workloads/synth.py
LAYER = (((4096, 4096), (1024, 4096), (1024, 4096)), ((4096, 4096),), ((14336, 4096), (14336, 4096)), ((4096, 14336),))


def listed():
    return [
        # the smallest stack of the benchmark: nothing but launch and latency
        {"name": "token_512x512", "kind": "token", "out": 512, "in": 512, "n": 4},
        # a key / value projection under a tight memory budget: few blocks loaded
        {"name": "token_1024x4096_n3", "kind": "token", "out": 1024, "in": 4096, "n": 3},
        # the benchmark's headline: an attention projection, one token
        {"name": "token_4096x4096", "kind": "token", "out": 4096, "in": 4096, "n": 16},
        # the MLP of a large model, one token: bound by the stream of the blocks
        {"name": "token_28672x8192", "kind": "token", "out": 28672, "in": 8192, "n": 16},
        # one token through a decoder layer: seven linears of different heights, launched from plans made once
        {"name": "layer_token", "kind": "layer", "n_lo": 8, "n_hi": 24, "slots": 24},
        # four sequences decoded together
        {"name": "batch4_14336x4096", "kind": "batch", "out": 14336, "in": 4096, "n": 16, "tokens": 4, "max_batch": 64},
        # sixteen sequences, the wide-input projection
        {"name": "batch16_4096x14336", "kind": "batch", "out": 4096, "in": 14336, "n": 16, "tokens": 16, "max_batch": 64},
        # odd sizes: a row count that is no multiple of any tile, a ragged batch, fp32 outputs
        {"name": "batch57_1056x2048_f32", "kind": "batch", "out": 1056, "in": 2048, "n": 5, "tokens": 57, "max_batch": 64, "f32": True},
        # a short prompt (ragged), no scratch lent
        {"name": "prompt300_14336x4096", "kind": "batch", "out": 14336, "in": 4096, "n": 16, "tokens": 300, "max_batch": 512},
        # a chunk of a prompt with the scratch buffer that all stacks of a model share
        {"name": "prompt1024_4096x14336", "kind": "batch", "out": 4096, "in": 14336, "n": 11, "tokens": 1024, "max_batch": 1024, "scratch": True},
        # a whole prompt through the largest stack, no scratch lent: the benchmark's prefill configuration
        {"name": "prompt2048_28672x8192", "kind": "batch", "out": 28672, "in": 8192, "n": 16, "tokens": 2048, "max_batch": 2048},
        # the other direction: a weight is decomposed into blocks on the device, packed, and restored to be checked
        {"name": "compress_4096x4096", "kind": "compress", "out": 4096, "in": 4096, "n": 2},
    ]


def _log_size(rng, lo, hi, step):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi))) / step)) * step))


def draw(rng):
    kind = rng.choice(("token", "token", "layer", "batch", "batch", "prompt", "prompt", "compress"))
    if kind == "layer":
        lo = rng.randint(1, 12)
        return {"kind": kind, "n_lo": lo, "n_hi": rng.randint(lo, 24), "slots": 24}
    if kind == "compress":
        return {"kind": kind, "out": _log_size(rng, 512, 4096, 32), "in": _log_size(rng, 512, 4096, 256), "n": rng.randint(1, 2)}
    while True:
        c = {"kind": "token" if kind == "token" else "batch", "out": _log_size(rng, 512, 28672, 32),
             "in": _log_size(rng, 512, 14336, 256), "n": rng.randint(1, 24)}
        if c["out"] * c["in"] * c["n"] <= 28672 * 8192 * 16:
            break
    if kind == "batch":
        c.update(tokens=_log_size(rng, 2, 64, 1), max_batch=64, f32=rng.random() < 0.25)
    elif kind == "prompt":
        tokens = _log_size(rng, 65, 2048, 1)
        c.update(tokens=tokens, max_batch=rng.choice((tokens, 2048)), f32=rng.random() < 0.25, scratch=rng.random() < 0.5)
    return c


def _generator(seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _scales(inn, seed):
    return np.exp(0.5 * np.random.default_rng(seed).standard_normal(inn)).astype(np.float32)


def _stack(out, inn, n, slots, max_batch, seed, g):
    """A stack with n loaded blocks like those of a decomposition: fair-coin signs; the leading factor columns positive and
    following the scales, the others zero-mean; magnitudes falling from block to block."""
    s = _scales(inn, seed)
    ps = B.PackedStack.empty(out, inn, slots, s, max_batch=max_batch, device=DEV)
    sn = torch.from_numpy(s / np.sqrt(np.mean(np.square(s, dtype=np.float64)))).to(DEV, torch.float32)
    shrink = (1024.0 / math.sqrt(float(out) * inn)) ** 0.25
    keep = []
    for i in range(n):
        lead, tail = 0.015 + 0.13 * math.exp(-i / 3.0), (0.0068 + 0.032 * math.exp(-i / 3.0)) * shrink
        words = torch.randint(-2**31, 2**31, (out, inn // 32), generator=g, device=DEV, dtype=torch.int64).to(torch.int32)
        u = tail * torch.randn((out, K), generator=g, device=DEV)
        v = tail * torch.randn((inn, K), generator=g, device=DEV)
        u[:, 0] = (lead * (1 + 0.08 * torch.randn(out, generator=g, device=DEV))).abs()
        v[:, 0] = (lead * (1 + 0.08 * torch.randn(inn, generator=g, device=DEV))).abs()
        v *= sn[:, None]
        u, v = u.half(), v.half()
        ps.push_block_device(words, u, v)
        keep.append((words, u, v))
    torch.cuda.synchronize()   # the canonical arrays are released on return
    return ps


def _activations(g, *shape):
    return torch.randn(shape, generator=g, device=DEV).half()


def prepare(case, seed):
    g = _generator(seed)
    kind = case["kind"]
    if kind == "compress":
        w = (0.02 * torch.randn((case["out"], case["in"]), generator=g, device=DEV)).half().float()
        return {"kind": kind, "w": w, "s": _scales(case["in"], seed), "n": case["n"]}
    if kind == "layer":
        heights = np.random.default_rng(seed).integers(case["n_lo"], case["n_hi"] + 1, size=7)
        keep, plans, ys, m = [], [], [], 0
        for group in LAYER:   # attention and activation functions come between the groups: a plan each
            x = _activations(g, group[0][1])
            items = []
            for out, inn in group:
                ps = _stack(out, inn, int(heights[m]), case["slots"], 1, seed + 1000 * m, g)
                y = torch.empty(out, dtype=torch.float16, device=DEV)
                items.append((x, ps, int(heights[m]), y))
                ys.append(y)
                m += 1
            keep.append(items)
            plans.append(B.TokenPlan(B.make_jobs(items)))
        return {"kind": kind, "plans": plans, "ys": ys, "keep": keep}
    out, inn, n = case["out"], case["in"], case["n"]
    if kind == "token":
        ps = _stack(out, inn, n, n, 1, seed, g)
        return {"kind": kind, "ps": ps, "n": n, "x": _activations(g, inn), "y": torch.empty(out, dtype=torch.float16, device=DEV)}
    ps = _stack(out, inn, n, n, case["max_batch"], seed, g)
    y = torch.empty((case["tokens"], out), dtype=torch.float32 if case.get("f32") else torch.float16, device=DEV)
    ws = torch.empty(B.dense_bytes(out, inn), dtype=torch.uint8, device=DEV) if case.get("scratch") else None
    return {"kind": kind, "ps": ps, "n": n, "x": _activations(g, case["tokens"], inn), "y": y, "ws": ws}


def run(state):
    kind = state["kind"]
    if kind == "token":
        return state["ps"].linear(state["x"], state["n"], state["y"])
    if kind == "layer":
        for plan in state["plans"]:
            plan.launch()
        return state["ys"]
    if kind == "compress":
        return B.PackedStack.from_dense(state["w"], state["s"], state["n"]).restore_weight(state["n"])
    if state["ws"] is not None:
        return state["ps"].linear_batched_ws(state["x"], state["n"], state["ws"], state["y"])
    return state["ps"].linear_batched(state["x"], state["n"], state["y"])


def work(case):
    """Bytes: the loaded blocks, scales and activations read once, the outputs written once.  Operations: rank-16 magnitudes times
    signs for every weight and block (as many in the factored form of one token), and a batch's product with the weight."""
    kind = case["kind"]
    if kind == "layer":
        mean = (case["n_lo"] + case["n_hi"]) / 2.0
        shapes = [s for group in LAYER for s in group]
        return {"bytes": sum(mean * B.block_bytes(o, i) + 2 * o for o, i in shapes) + sum(6 * g[0][1] for g in LAYER),
                "flops": sum(mean * 2.0 * K * o * i for o, i in shapes)}
    out, inn, n = case["out"], case["in"], case["n"]
    if kind == "compress":
        # the weight in, the blocks and the restored weight out; 16 rounds of two products with 32 columns per block
        return {"bytes": 4.0 * out * inn + 2.0 * n * B.block_bytes(out, inn) + 2.0 * out * inn,
                "flops": n * (16 * 2 * 2.0 * 32 + 2.0 * 2 * K) * out * inn}
    tokens = case.get("tokens", 1)
    return {"bytes": n * B.block_bytes(out, inn) + 4.0 * inn + 2.0 * tokens * inn + (4.0 if case.get("f32") else 2.0) * tokens * out,
            "flops": 2.0 * K * n * out * inn + (2.0 * tokens * out * inn if tokens > 1 else 0.0)}


def tolerance(case):
    if case["kind"] == "compress":
        # four times what a relative change of the weight by 1e-7 does to the restored weight (5.4e-3): residuals near zero take
        # the other sign, and the bf16 iterates of the subspace rounds turn with it.  Single weights may differ by a whole sign.
        return {"rel": 2e-2}
    # four times the path's distance to an evaluation in 64 bits: 2.9e-4 to 4.3e-4 (fp16 weights or panels and fp16 outputs),
    # largest 1.1e-3 to 1.8e-3
    return {"rel": 1.6e-3, "max": 7e-3}
