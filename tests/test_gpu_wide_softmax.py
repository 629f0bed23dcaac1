"""Softmax and its backward for windows beyond 13 (na2d_generic.hip): rows of one wave and of four, at both ends of each
number of elements a lane keeps; in place; and 16-bit rows against fp32 rows in time."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import synth
from gpu_util import assert_close, to_np

pytestmark = pytest.mark.gpu


def _rows(H, W, k, dtype, seed):
    rng = np.random.RandomState(seed)
    shape = (1, 1, H, W, k * k)
    like = torch.empty((1, 1, H, W, 32), dtype=synth.TORCH_DTYPES[dtype], device="cuda")
    return like, *(synth.to_device(synth.round_to(rng.randn(*shape).astype(np.float32), dtype), dtype) for _ in range(2))


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("k", [15, 17, 21, 23, 31, 33, 45, 47, 63])
def test_softmax_of_wide_windows(oracle, k, dtype):
    like, logits, dp = _rows(k, k + 2, k, dtype, seed=k)   # (the number of rows is no multiple of four: k and k + 2 are odd)
    attn = na.na2d_softmax(logits, k, like, torch.empty_like(logits))
    assert_close("softmax", attn, oracle.softmax(to_np(logits)), dtype)
    ds = na.na2d_softmax_bwd(attn, dp, k, like, torch.empty_like(dp))
    want = oracle.softmax_bwd(to_np(attn), to_np(dp))
    assert_close("softmax backward", ds, want, dtype)
    # the weights are small: hold ds to its own size too (one rounding of the result, and the dot product in fp32)
    ulp = {"f32": 2.0 ** -19, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[dtype]
    small = 2.0 ** -24 if dtype == "f16" else 0.0
    a = to_np(attn)
    assert np.all(np.abs(to_np(ds) - want) <= small + ulp * a * (np.abs(to_np(dp)) + np.abs((a * to_np(dp)).sum(-1, keepdims=True)) + 1e-2))
    na.na2d_softmax(logits, k, like, logits)
    na.na2d_softmax_bwd(attn, dp, k, like, dp)
    assert torch.equal(logits, attn) and torch.equal(dp, ds)


@pytest.mark.parametrize("k", [31, 45, 63])
def test_sixteen_bit_rows_take_no_longer_than_fp32_rows(k):
    # half the bytes: a row whose loads wait for each other, or that leaves a few waves in flight, shows as the slower one
    def best(dtype):
        like, p, dp = _rows(70, 63, k, dtype, seed=1)
        ds, times = torch.empty_like(dp), []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(10):
                na.na2d_softmax_bwd(p, dp, k, like, ds)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    assert best("f16") <= 1.15 * best("f32")
