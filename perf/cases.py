"""What is timed: the products and block selections a user of this library has it do.

A case is a dict of plain values.  kind "product": Y = act(W X + bias) of one pruned layer through spmm /
spmm_fused on a packed handle that the program keeps; kind "select": the block list of one dense layer
through select_blocks, which works on host arrays by its nature.

Sizes: the layers of synthetic/configs.py (c0 .. c4 and the paper's block shapes n1 .. n4), the same layers at
batch 1 (7 x 7 and 14 x 14 maps: 49 and 196 pixels, rows of X that are not 16-byte aligned), and a fully
connected layer on a small batch.  X and Y are contiguous, as an allocator gives them.
"""
import math

import numpy as np
import torch

import paper_2407_19644_amd as ubp

TORCH = {"f32": torch.float32, "f16": torch.float16, "bf16": torch.bfloat16}
BYTES = {"f32": 4, "f16": 2, "bf16": 2}


def product(name, M, K, N, bh, bw, density, dtype, y_dtype=None, mask="uniform", act="none"):
    c = {"kind": "product", "M": M, "K": K, "N": N, "bh": bh, "bw": bw, "density": density, "dtype": dtype,
         "y_dtype": y_dtype or dtype, "mask": mask, "act": act}
    return dict(c, name=name) if name else c


def listed():
    return [
        # c0: one 14 x 14 map through a tiny fp32 layer; the smallest call there is
        product("tiny_f32", 64, 64, 196, 4, 4, 0.5, "f32"),
        # c1's layer for a single image (7 x 7), with its bias and a clamp to [0, 6]: latency of one pointwise convolution, odd rows
        product("pointwise_b1", 960, 160, 49, 4, 4, 0.3, "f16", act="clamp"),
        # n2's layer for a single image (14 x 14): 4 x 1 blocks, rows of 392 bytes
        product("pointwise512_b1", 512, 512, 196, 4, 1, 0.2, "f16", mask="columns"),
        # a fully connected layer on a batch of 16: c4's weights without the skew, hardly any pixels
        product("fc_b16", 4096, 4096, 16, 16, 16, 0.1, "bf16"),
        # c1's layer at batch 64
        product("pointwise_b64", 960, 160, 3136, 4, 4, 0.3, "f16"),
        # n3: tall one-column blocks at 90 % sparsity, read back in fp32
        product("pointwise1024_b32", 1024, 1024, 1568, 8, 1, 0.1, "f16", y_dtype="f32", mask="columns"),
        # an fp32 layer of ordinary size (n2's, batch 32)
        product("pointwise512_f32_b32", 512, 512, 6272, 4, 1, 0.2, "f32", mask="columns"),
        # c2: 1 x 1 expand convolution at batch 64
        product("expand_b64", 1024, 256, 12544, 8, 8, 0.2, "f16"),
        # n4: 3 x 3 convolution through im2col, blocks of 4 channels x (3 x 3), with bias and ReLU, batch 32
        product("conv3x3_b32", 256, 2304, 6272, 4, 9, 0.2, "bf16", mask="columns", act="relu"),
        # c3: 3 x 3 convolution through im2col, square blocks, batch 64
        product("conv3x3_b64", 256, 2304, 12544, 4, 4, 0.25, "bf16"),
        # c4: the largest layer, skewed block counts per stripe
        product("stress", 4096, 4096, 8192, 16, 16, 0.1, "bf16", mask="zipf"),
        # choosing the blocks of a pointwise layer (expansion and division), once per layer and pruning step
        {"name": "select_bed", "kind": "select", "M": 512, "K": 512, "bh": 4, "bw": 1, "density": 0.2, "dtype": "f16",
         "method": "bed", "aligned": False},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _channels(rng, lo, hi):
    """A channel count: mostly a multiple of 8, as networks have them, sometimes any number (pruned channels)."""
    n = _log(rng, lo, hi)
    return n if rng.random() < 0.3 else max(8, 8 * round(n / 8))


def _pixels(rng, most):
    """Pixels x batch of a 7 x 7 .. 56 x 56 map."""
    side = rng.choice([s for s in (7, 14, 28, 56) if s * s <= most])
    return side * side * _log(rng, 1, max(1, min(64, most // (side * side))))


def draw(rng):
    family = rng.choice(("pointwise", "pointwise", "square", "square", "conv", "conv", "blocks16", "blocks16", "fc", "f32", "select"))
    act = rng.choice(("none", "none", "relu", "clamp"))
    half = rng.choice(("f16", "bf16"))
    y = rng.choice((half, half, half, "f32"))
    if family == "pointwise":       # N x 1 blocks
        bh, d = rng.choice(((2, 0.3), (4, 0.2), (8, 0.1), (4, 0.3), (16, 0.2)))
        return product(None, _channels(rng, 64, 1024), _channels(rng, 32, 1024), _pixels(rng, 25088), bh, 1, d, half, y, "columns", act)
    if family == "square":          # small square blocks on 1 x 1 convolutions
        b, d = rng.choice(((4, 0.3), (8, 0.2), (4, 0.15), (8, 0.3)))
        return product(None, _channels(rng, 64, 1024), _channels(rng, 32, 1024), _pixels(rng, 12544), b, b, d, half, y, "uniform", act)
    if family == "conv":            # 3 x 3 convolutions through im2col
        K = 9 * _channels(rng, 32, 256)
        if rng.random() < 0.5:
            return product(None, _channels(rng, 64, 512), K, _pixels(rng, 12544), rng.choice((2, 4, 8)), 9, rng.choice((0.2, 0.3)), half, y, "columns", act)
        return product(None, _channels(rng, 64, 512), K, _pixels(rng, 12544), 4, 4, rng.choice((0.15, 0.25)), half, y, "uniform", act)
    if family == "blocks16":        # large layers of 16 x 16 blocks, even or skewed
        N = _log(rng, 64, 8192 if y != "f32" else 4096)
        return product(None, 16 * _log(rng, 32, 256), 16 * _log(rng, 72, 256), N if rng.random() < 0.4 else 64 * round(N / 64), 16, 16,
                       rng.choice((0.05, 0.1)), half, y, rng.choice(("uniform", "zipf")), act)
    if family == "fc":              # fully connected layers on small batches
        b, d = rng.choice(((4, 0.2), (8, 0.2), (16, 0.1), (16, 0.2)))
        return product(None, _channels(rng, 512, 4096), _channels(rng, 512, 4096), _log(rng, 1, 64), b, b, d, half, y, "uniform", act)
    if family == "f32":
        bh, bw, d, mask = rng.choice(((4, 4, 0.3, "uniform"), (8, 8, 0.2, "uniform"), (4, 1, 0.2, "columns"), (2, 1, 0.3, "columns"), (16, 16, 0.1, "uniform")))
        return product(None, _channels(rng, 64, 1024), _channels(rng, 64, 1024), _pixels(rng, 6272), bh, bw, d, "f32", "f32", mask, act)
    return {"kind": "select", "M": _channels(rng, 64, 1024), "K": _channels(rng, 64, 512), "bh": rng.choice((2, 4, 8)), "bw": rng.choice((1, 1, 4)),
            "density": rng.choice((0.1, 0.2, 0.3)), "dtype": rng.choice(("f32", "f16", "bf16")), "method": rng.choice(("greedy", "bed", "bed")),
            "aligned": rng.random() < 0.2}


def _count(case):
    return ubp.target_block_count(case["M"], case["K"], case["bh"], case["bw"], case["density"])


def _blocks(case, seed):
    """A valid unaligned block list."""
    M, K, bh, bw = case["M"], case["K"], case["bh"], case["bw"]
    if case["mask"] != "columns":
        return ubp.select_reference(M, K, bh, bw, case["density"], seed, 1 if case["mask"] == "zipf" else 0, 1.1)
    # the paper's blocks: bh consecutive output channels of one column group, rows anywhere.  Blocks per group
    # as even as the count allows; k starts without overlap = k different numbers below M - k (bh - 1), sorted, spread apart.
    rng = np.random.default_rng(seed)
    groups = K // bw
    per = np.full(groups, _count(case) // groups)
    per[rng.permutation(groups)[:_count(case) - int(per.sum())]] += 1
    out = []
    for g in range(groups):
        k = min(int(per[g]), M // bh)
        r = np.sort(rng.choice(M - k * (bh - 1), size=k, replace=False)) + np.arange(k) * (bh - 1)
        out.append(np.stack([r, np.full(k, g * bw)], axis=1))
    return np.concatenate(out).astype(np.int32)


def _to_numpy(t):
    t = t.cpu()
    return t.view(torch.int16).numpy().view(np.uint16) if t.dtype == torch.bfloat16 else t.numpy()


def prepare(case, seed):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    M, K, dtype = case["M"], case["K"], case["dtype"]
    # trained weights: He scale, some output channels more important than others where blocks are chosen by magnitude
    W = torch.randn(M, K, generator=gen, device="cuda") * math.sqrt(2.0 / K)
    if case["kind"] == "select":
        W = W * torch.exp(0.5 * torch.randn(M, 1, generator=gen, device="cuda"))
        return {"case": case, "W": _to_numpy(W.to(TORCH[dtype]))}
    N, y_dtype = case["N"], case["y_dtype"]
    packed = ubp.pack(_to_numpy(W.to(TORCH[dtype])), dtype, case["bh"], case["bw"], _blocks(case, seed), device=torch.cuda.current_device())
    # activations after a ReLU; the stress layer's kind (16 x 16 blocks) and fully connected inputs are plain normal
    X = torch.randn(K, N, generator=gen, device="cuda")
    if case["bh"] < 16:
        X = X.relu_()
    X = X.to(TORCH[dtype])
    Y = torch.empty(M, N, dtype=TORCH[y_dtype], device="cuda")
    bias = 0.5 * torch.randn(M, generator=gen, device="cuda") if case["act"] != "none" else None
    ubp.spmm_prepare(packed, X.data_ptr(), N, N, Y.data_ptr(), N, y_dtype)
    return {"case": case, "packed": packed, "X": X, "Y": Y, "bias": bias, "N": N, "y_dtype": y_dtype, "act": case["act"]}


def run(state):
    if "W" in state:
        c = state["case"]
        return ubp.select_blocks(state["W"], c["dtype"], c["bh"], c["bw"], c["density"], c["method"], c["aligned"])
    X, Y, N = state["X"], state["Y"], state["N"]
    stream = torch.cuda.current_stream().cuda_stream
    if state["bias"] is None:
        ubp.spmm(state["packed"], X.data_ptr(), N, N, Y.data_ptr(), N, state["y_dtype"], stream)
    else:
        ubp.spmm_fused(state["packed"], X.data_ptr(), N, N, Y.data_ptr(), N, state["y_dtype"], state["bias"].data_ptr(), state["act"], 0.0, 6.0,
                       stream)
    return Y


def work(case):
    M, K, bh, bw, nb, esz = case["M"], case["K"], case["bh"], case["bw"], _count(case), BYTES[case["dtype"]]
    if case["kind"] == "select":    # every weight read and added once, the block list written
        return {"bytes": M * K * esz + 8 * nb, "flops": M * K}
    N = case["N"]
    weights = nb * bh * bw * esz + (M - bh + 2) * 4 + nb * 4
    return {"bytes": weights + K * N * esz + M * N * BYTES[case["y_dtype"]] + (4 * M if case["act"] != "none" else 0),
            "flops": 2 * nb * bh * bw * N}


def tolerance(case):
    if case["kind"] == "select":
        return "exact"
    # fp32 sums everywhere; a 16-bit Y is rounded once, where two orders of addition may fall on different sides
    return {"f32": {"rel": 1e-5, "max": 1e-4}, "f16": {"rel": 5e-4, "max": 2e-3}, "bf16": {"rel": 4e-3, "max": 1.6e-2}}[case["y_dtype"]]
