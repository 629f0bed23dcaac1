"""The fused forward over 4 x 4 patches against the oracle: remainders of patches, tiles and streamed rows, with one, two, four and eight waves to
a patch, with a running maximum that rises from row to row, and one that starts at -inf."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_util import Stages, assert_close
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth

pytestmark = pytest.mark.gpu


def check(oracle, p, host, use_rpb=True, planes=(0, -1), scale=None):
    st = Stages(p, host, use_rpb=use_rpb, scale=scale)
    st.forward_fused()
    for b in planes:
        q, k, v = (host[n][b:][:1].astype(np.float64) for n in ("q", "k", "v"))
        out, lse = oracle.fwd(q, k, v, host["rpb"].astype(np.float64) if use_rpb else None, st.scale, p.k, return_lse=True)
        assert_close("out", st.out_fused[b:][:1], out, p.dtype)
        assert_close("lse", st.lse[b:][:1], lse, "f32")


# 16 .. 24, 180 .. 240, 960 .. 1300 and 3000 and more patches: eight, four, two waves to a patch and one; k = 3 has rows of blocks for two only
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("B,H,W,D,k", [
    (1, 17, 15, 32, 15), (1, 21, 22, 16, 21), (10, 17, 15, 32, 15), (5, 23, 26, 64, 17), (3, 35, 34, 16, 31), (40, 17, 22, 32, 15), (170, 17, 15, 32, 15),
    (120, 22, 18, 64, 17), (2, 16, 13, 128, 13), (12, 17, 15, 128, 15), (130, 13, 21, 128, 13)])
def test_patches_shared_by_waves(oracle, dtype, B, H, W, D, k):
    p = synth.Problem(B, 1, H, W, D, k, dtype)
    check(oracle, p, synth.make_inputs(p, seed=H * W + B, rpb_std=0.5), use_rpb=(B != 5))


@pytest.mark.parametrize("B,H,W,D,k", [(1, 3, 3, 32, 3), (1, 5, 7, 64, 5), (20, 9, 10, 32, 9), (200, 14, 14, 32, 7), (64, 7, 33, 32, 7), (40, 30, 9, 64, 3), (60, 29, 11, 16, 11), (4, 12, 40, 128, 5)])
def test_narrow_windows_in_fp32(oracle, B, H, W, D, k):
    p = synth.Problem(B, 1, H, W, D, k, "f32")
    check(oracle, p, synth.make_inputs(p, seed=H + W + B, rpb_std=0.5), use_rpb=(k != 9))


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("B", [1, 30, 200])
def test_maximum_that_moves(oracle, dtype, B):
    """A bias that rises (and, in a second head, falls) from row to row (in fp32 by little: the spacing of a logit of 50 is 4e-6): the base of the weights moves in every row of blocks, or in none but the
    first.  A third head starts with rows of -inf."""
    H, W, D, k = 19, 18, 32, 17
    p = synth.Problem(B, 3, H, W, D, k, dtype)
    host = synth.make_inputs(p, seed=B)
    rise = np.arange(2 * k - 1, dtype=np.float32)[:, None] * (1.5 if dtype == "f32" else 12.0)
    host["rpb"][0] = rise
    host["rpb"][1] = -rise
    host["rpb"][2, : k - 3] = -np.inf
    check(oracle, p, host, planes=(0,), scale=0.05)


@pytest.mark.parametrize("planes", [1, 100])   # eight waves to a patch and one
def test_smallest_fp16_weights(planes):
    """One key takes all but 2^-27 of a query's weight and has no value; the others weigh 3 * 2^-39 of it each, which fp16 holds exactly once the largest is
    2^15: with one bit less the output would be a third too large."""
    H, W, D, k = 62, 31, 16, 31
    q, key, v = (torch.zeros(planes, 1, H, W, D, dtype=torch.float16, device="cuda") for _ in range(3))
    v[..., 1::2, :] = 6e4
    rpb = torch.zeros(1, 2 * k - 1, 2 * k - 1, dtype=torch.float16, device="cuda")
    rpb[:, k - 1, k - 1] = 39 * np.log(2) - np.log(3)   # (to 2^-7: the weights to 0.8 %)
    out = F.na2d(q, key, v, rpb, kernel_size=k)[..., 0::2, :].double()
    large = k * (torch.arange(k).remainder(2) == 1).sum().item()   # (W = k: every window holds all columns)
    p = torch.exp(-rpb[0, k - 1, k - 1].double())
    want = large * p * v[0, 0, 0, 1, 0].double() / (1 + (k * k - 1) * p)
    assert W == k and (out / want - 1).abs().max() < 0.02
