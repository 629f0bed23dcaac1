"""What this library is timed on: neighbourhood attention as a program calls it, through ``functional``.

A case is one call (inference), or one forward and backward pass (training), of the 2D or the 1D operator on inputs
that lie on the GPU.  The sizes are those of the workload table (``synth.CONFIGS``, ``synth.CONFIGS_1D``), of the
kernel-size study (k = 3 .. 13) and of the parity tests (odd map sides, other head dims, windows beyond 13).
"""
from __future__ import annotations

import math

import torch

from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd.synth import TORCH_DTYPES


def _map(name, op, B, heads, H, W, D, k, dtype, bias=True):
    return {"name": name, "op": op, "B": B, "heads": heads, "H": H, "W": W, "D": D, "k": k, "dtype": dtype, "bias": bias}


def _seq(name, op, B, heads, L, k, dtype):
    return {"name": name, "op": op, "B": B, "heads": heads, "H": 1, "W": L, "D": 32, "k": k, "dtype": dtype, "bias": True}


def listed():
    return [
        # serving one 224 x 224 image: a layer of the third stage, where most of the model's layers are (latency)
        _map("infer_one_image_stage3_f16", "infer", 1, 8, 14, 14, 32, 7, "f16"),
        # the first layers of a detector on an 800 x 1333 image: a large map, a small batch
        _map("infer_detection_f16", "infer", 2, 2, 200, 334, 32, 7, "f16"),
        # training the classifier: first stage (the benchmark's shape), one fused forward and one fused backward
        _map("train_stage1_f16", "train", 64, 2, 56, 56, 32, 7, "f16"),
        # ... and the third stage: small maps, many planes
        _map("train_stage3_bf16", "train", 128, 8, 14, 14, 32, 7, "bf16"),
        # the same first stage as the paper composes it: logits, softmax and weighted sum as differentiable steps
        _map("train_unfused_stage1_f16", "unfused", 64, 2, 56, 56, 32, 7, "f16"),
        # the largest window of the kernel-size study
        _map("train_stage1_k13_f16", "train", 64, 2, 56, 56, 32, 13, "f16"),
        # full precision training (no mixed precision)
        _map("train_stage1_f32", "train", 64, 2, 56, 56, 32, 7, "f32"),
        # the first stage's 64 channels as one head
        _map("train_head_dim_64_f16", "train", 64, 1, 56, 56, 64, 7, "f16"),
        # odd sizes: a map that no tile divides, 16-channel heads, a small window, no bias table
        _map("train_ragged_no_bias_bf16", "train", 5, 3, 61, 45, 16, 5, "bf16", bias=False),
        # a window beyond the study's, on a small batch
        _map("train_wide_window_k21_bf16", "train", 4, 2, 64, 64, 32, 21, "bf16"),
        # 1D: the first stage's tokens as sequences
        _seq("train_sequence_k7_f16", "train1d", 64, 2, 3136, 7, "f16"),
        _seq("infer_sequence_k31_bf16", "infer1d", 64, 2, 3136, 31, "bf16"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


# A drawn case takes at most this many (query, key) products per contraction and this many elements in each of q, k, v:
# those of the first stage at k = 7, and for windows beyond 13 a quarter of the products of the listed one.
_MOST_ELEMENTS = 64 * 2 * 56 * 56 * 32
_MOST_PRODUCTS = _MOST_ELEMENTS * 49
_MOST_PRODUCTS_WIDE = 4 * 2 * 64 * 64 * 32 * 441 // 4


def draw(rng):
    op = rng.choice(["infer", "infer", "train", "train", "train", "unfused", "infer1d", "train1d"])
    dtype = rng.choice(["f16", "f16", "bf16", "bf16", "f32"])
    bias = rng.random() < 0.8
    heads = rng.choice([1, 2, 3, 4, 6, 8, 16])
    if op.endswith("1d"):
        D, k = 32, rng.choice([3, 5, 7, 7, 9, 13, 21, 31, 63])
        H, W = 1, _log_uniform(rng, max(k, 64), 16384)
        window = k
    else:
        D = rng.choice([32, 32, 32, 32, 16, 64, 128])
        k = rng.choice([3, 5, 7, 7, 7, 9, 11, 13, rng.choice([15, 17, 21, 25, 31])])
        H = _log_uniform(rng, max(k, 7), 256)
        W = min(384, max(k, 7, int(round(H * math.exp(rng.uniform(-0.7, 0.7))))))
        window = k * k

    def most_items():
        positions = heads * H * W
        products = _MOST_PRODUCTS if H == 1 or k <= 13 else _MOST_PRODUCTS_WIDE
        return min(_MOST_ELEMENTS // (positions * D), products // (positions * max(D, 32) * window))

    while most_items() < 1:   # one item is already more than that: fewer heads, then a smaller map, then fewer channels
        if heads > 1:
            heads //= 2
        elif max(H, W) > k:
            H, W = (1, max(k, W // 2)) if H == 1 else (max(k, H // 2), max(k, W // 2))
        else:
            D //= 2
    B = _log_uniform(rng, 1, most_items())
    return {"op": op, "B": B, "heads": heads, "H": H, "W": W, "D": D, "k": k, "dtype": dtype, "bias": bias}


def _is_1d(case):
    return case["op"].endswith("1d")


def prepare(case, seed):
    """Activations of unit variance and a small bias table in the case's dtype, as after a normalisation and a
    projection; for training the leaves carry gradients and the upstream gradient is in hand."""
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = TORCH_DTYPES[case["dtype"]]
    k, train = case["k"], not case["op"].startswith("infer")
    space = (case["W"],) if _is_1d(case) else (case["H"], case["W"])
    shape = (case["B"], case["heads"], *space, case["D"])
    normal = lambda s, std=1.0: torch.randn(s, generator=g, device="cuda", dtype=torch.float32).mul_(std).to(dt)
    q, key, v = (normal(shape).requires_grad_(train) for _ in range(3))
    table = (case["heads"],) + (2 * k - 1,) * len(space)
    rpb = normal(table, 0.02).requires_grad_(train) if case["bias"] else None
    dout = normal(shape) if train else None
    op = {"infer": F.na2d, "train": F.na2d, "unfused": F.na2d_unfused, "infer1d": F.na1d, "train1d": F.na1d}[case["op"]]
    return {"op": op, "q": q, "k": key, "v": v, "rpb": rpb, "dout": dout, "kernel_size": k}


def run(state):
    q, k, v, rpb, dout = (state[n] for n in ("q", "k", "v", "rpb", "dout"))
    if dout is None:
        with torch.no_grad():
            return state["op"](q, k, v, rpb, kernel_size=state["kernel_size"])
    out = state["op"](q, k, v, rpb, kernel_size=state["kernel_size"])
    leaves = (q, k, v) if rpb is None else (q, k, v, rpb)
    return (out.detach(), *torch.autograd.grad(out, leaves, dout))


def _gather_indices(case):
    """For each window slot: the flat key position of every query and the flat cell of the bias table it uses."""
    k, dev = case["k"], "cuda"

    def axis(length, window):
        pos = torch.arange(length, device=dev)
        first = (pos - (window - 1) // 2).clamp(0, length - window)
        return [(first + a, first + a - pos + window - 1) for a in range(window)]

    cells = 2 * k - 1
    for y, cy in axis(case["H"], 1 if _is_1d(case) else k):
        for x, cx in axis(case["W"], k):
            yield (y[:, None] * case["W"] + x).flatten(), (cy[:, None] * cells + cx).flatten()


def exact(case, seed):
    """The operator and its chain rule in 64 bits, one window slot at a time."""
    state = prepare(case, seed)
    B, heads, D, n = case["B"], case["heads"], case["D"], case["H"] * case["W"]
    wide = lambda t: t.detach().double()
    flat = lambda t: wide(t).reshape(B, heads, n, D)
    shaped = state["q"].shape
    q, key, v = (flat(state[name]) for name in ("q", "k", "v"))
    scale = float(D) ** -0.5
    slots = list(_gather_indices(case))
    table = wide(state["rpb"]).flatten(1) if case["bias"] else None
    logits = torch.stack([(q * key[:, :, at]).sum(-1).mul_(scale) + (0 if table is None else table[:, cell])
                          for at, cell in slots])
    p = torch.softmax(logits, 0)
    out = sum(p[s].unsqueeze(-1) * v[:, :, at] for s, (at, _) in enumerate(slots))
    if state["dout"] is None:
        return out.reshape(shaped)
    dout = flat(state["dout"])
    dp = torch.stack([(dout * v[:, :, at]).sum(-1) for at, _ in slots])
    ds = p * (dp - (p * dp).sum(0))
    dq, dk, dv = (torch.zeros_like(q) for _ in range(3))
    dtable = None if table is None else torch.zeros_like(table)
    for s, (at, cell) in enumerate(slots):
        w = ds[s].unsqueeze(-1)
        dq += w * key[:, :, at]
        dk.index_add_(2, at, w * q)
        dv.index_add_(2, at, p[s].unsqueeze(-1) * dout)
        if dtable is not None:
            dtable.index_add_(1, cell, ds[s].sum(0))
    grads = [t.mul_(f).reshape(shaped) for t, f in ((dq, scale), (dk, scale), (dv, 1.0))]
    return (out.reshape(shaped), *grads) + (() if dtable is None else (dtable.reshape(state["rpb"].shape),))


def work(case):
    """q, k, v (and the upstream gradient) read once, the output (and three gradients) written once, the bias table
    (and its gradient); two contractions forward, four backward, over every (query, key) pair of a window."""
    e = 4 if case["dtype"] == "f32" else 2
    window = case["k"] if _is_1d(case) else case["k"] ** 2
    table = (2 * case["k"] - 1) ** (1 if _is_1d(case) else 2) * case["heads"] * e if case["bias"] else 0
    n = case["B"] * case["heads"] * case["H"] * case["W"] * case["D"]
    train = not case["op"].startswith("infer")
    return {"bytes": (8 if train else 4) * n * e + (2 if train else 1) * table, "flops": (12 if train else 4) * n * window}


def tolerance(case):
    """Relative 2-norm, about four times the distance from the same operator in 64 bits: one rounding to the storage
    type in the fused operators' outputs; the weights and their gradients rounded once more wherever the backward runs
    in separate steps; the logits too in the unfused forward."""
    if case["op"].startswith("infer"):
        return {"rel": {"f32": 2e-6, "f16": 1e-3, "bf16": 7e-3}[case["dtype"]]}
    return {"rel": {"f32": 8e-6, "f16": 2.5e-3, "bf16": 2e-2}[case["dtype"]]}
