"""Both sides of the rules by which a 2D problem takes the plain-ALU tiles (fp32), strips shared by four waves or strips of
one wave each, and the instances that only wide windows reach: every stage, forward and backward, against the oracle."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from gpu_util import assert_close
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth
from test_gpu_parity import run_all

pytestmark = pytest.mark.gpu


def _some_planes(p):
    return [(b, h) for b in sorted({0, p.B // 2, p.B - 1}) for h in range(p.heads)]


# 1254, 1311, 1539 and 6156 strips on maps of three to a row (below 1280 no fp32 problem runs in tiles, from there logits and
# fused forward of small windows do, from 1536 on wider ones and weighted sums, from 6144 on whatever has tiles), 3066 and 4116
# on maps of one (logits from 2560 on, weighted sums from 3072, inverse sums from 4096)
@pytest.mark.parametrize("H,W,B", [(19, 37, 22), (19, 37, 23), (19, 37, 27), (19, 37, 108), (21, 13, 146), (21, 13, 196)])
@pytest.mark.parametrize("D,k", [(16, 3), (16, 5), (16, 7), (16, 9), (16, 11), (32, 3), (32, 5), (32, 7), (64, 3), (64, 5)])
def test_fp32_tiles_and_strips(oracle, D, k, H, W, B):
    # maps that no tile and no strip divides; per head dim the widest window that each operator's tiles take, and those in
    # between where only some of the operators do
    p = synth.Problem(B, 1, H, W, D, k, "f32")
    run_all(oracle, p, seed=B + D + k, planes=_some_planes(p), use_rpb=(k != 9), rpb_std=0.5)


def test_fp32_rows_shorter_than_a_strip():
    # as many queries on 7 x 7 maps make twice as many strips, and in a call of this size the tiles hide their empty lanes:
    # the fused forward must not take twice the time there (kernels alone, out of a graph of 20 calls)
    def best(B, H, W):
        q, key, v = (torch.randn(B, 1, H, W, 16, device="cuda") for _ in range(3))
        out, graph, times = torch.empty_like(q), torch.cuda.CUDAGraph(), []
        call = lambda: na.na2d_fused_fwd(q, key, v, None, 0.25, 5, out)
        call()
        torch.cuda.synchronize()
        with torch.cuda.graph(graph):
            for _ in range(20):
                call()
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)
    assert best(458, 7, 7) <= 1.25 * best(28, 28, 28)   # (strips / strips 1.5, tiles / tiles 0.95)


# The strips (planes x H x ceil(W / 16)) from which on a wave of the logits keeps one to itself (k <= 5 at D = 128, what has no tiles there, D >= 64 to
# k = 13), and the same numbers for heads and windows whose logits stay with four.  (The fused forward of these problems runs over patches; where
# it still takes strips: test_fused_forward_in_strips.)  H is no multiple of the four strips of a workgroup; W leaves 0, 1, 2 or 15
# positions in a row's last strip.
@pytest.mark.parametrize("H,W,D,k,dtype,strips", [
    (5, 16, 128, 3, "f32", 1536), (6, 17, 64, 5, "f32", 1536), (7, 15, 64, 5, "f32", 3584),
    (13, 17, 32, 9, "f32", 6144), (14, 31, 128, 9, "f32", 6144), (15, 16, 128, 9, "f16", 6144),
    (13, 33, 128, 13, "f16", 6144), (14, 18, 128, 13, "bf16", 6144), (11, 17, 64, 11, "f32", 6144),
    (17, 18, 32, 15, "bf16", 12288), (15, 31, 16, 15, "f16", 12288), (15, 16, 64, 15, "f32", 12288),
])
@pytest.mark.parametrize("above", [False, True])
def test_strips_of_four_waves_and_of_one(oracle, H, W, D, k, dtype, strips, above):
    per_plane = H * ((W + 15) // 16)
    p = synth.Problem((strips + per_plane - 1) // per_plane - (0 if above else 1), 1, H, W, D, k, dtype)
    run_all(oracle, p, seed=H * W + k, planes=_some_planes(p), rpb_std=0.5)


@pytest.mark.parametrize("B", [46, 47])   # 32338 and 33041 queries; from 32768 on 128 channels are summed slice by slice
@pytest.mark.parametrize("k,dtype", [(3, "f16"), (5, "bf16"), (7, "f16"), (9, "bf16"), (13, "f16")])
def test_four_slices_and_strips(oracle, k, dtype, B):
    p = synth.Problem(B, 1, 19, 37, 128, k, dtype)
    run_all(oracle, p, seed=B + k, planes=_some_planes(p), rpb_std=0.5, e2e_unfused=False)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("heads,H,W,D,k", [
    (2, 15, 16, 32, 15), (2, 17, 33, 16, 17), (2, 19, 19, 64, 19), (2, 13, 31, 128, 13),   # the strips' edges
    # as many positions as the windows reach, a strip more, and the softmax instances of k = 23 .. 31, 33 .. 45, 47 .. 63
    (2, 23, 47, 32, 23), (2, 31, 33, 16, 31), (1, 34, 49, 32, 33), (1, 45, 47, 64, 45), (1, 63, 65, 16, 63), (1, 25, 40, 128, 25),
])
def test_wide_windows_forward_and_backward(oracle, heads, H, W, D, k, dtype):
    run_all(oracle, synth.Problem(1, heads, H, W, D, k, dtype), seed=H * W + D + k, rpb_std=0.5)


def test_more_strips_than_a_launch_holds():
    # 16.8 million strips (more than 2^32 threads) on 3 x 3 maps, where every query sees every key: slot = key
    B, D = 5592500, 32
    gen = torch.Generator(device="cuda").manual_seed(7)
    attn = torch.rand(B, 1, 3, 3, 9, device="cuda", generator=gen)
    dout = torch.rand(B, 1, 3, 3, D, device="cuda", generator=gen)
    dv = torch.full_like(dout, float("nan"))
    na.na2d_av_bwd_v(attn, dout, 3, dv)
    assert not torch.isnan(dv).any()
    for first in (0, B // 2, 5592380, B - 64):   # (a launch holds 5592400 planes)
        part = slice(first, first + 64)
        a, x = attn[part].double().cpu().view(64, 9, 9), dout[part].double().cpu().view(64, 9, D)
        want = (a.unsqueeze(-1) * x.unsqueeze(2)).sum(1)
        # nine products of numbers below 1, added in fp32
        torch.testing.assert_close(dv[part].double().cpu().view(64, 9, D), want, rtol=0, atol=9 * 9 * 2.0 ** -24)


class _Problem(ctypes.Structure):   # as the library's launch functions take it
    _fields_ = [(n, ctypes.c_int) for n in ("B", "heads", "H", "W", "K", "dtype", "D")]


def _fused_runs_in_strips(p):
    q = ctypes.byref(_Problem(p.B, p.heads, p.H, p.W, p.k, {"f32": 0, "f16": 1, "bf16": 2}[p.dtype], p.D))
    asked = [getattr(na.load(), n) for n in ("_ZN4na2d20fused_mfma_supportedERKNS_7ProblemE", "_ZN4na2d19patch_fwd_preferredERKNS_7ProblemE")]
    for f in asked:
        f.restype = ctypes.c_bool
    return not any(f(q) for f in asked) and p.D * p.k > 7 * 16   # (none of these has tiles)


# Where the fused forward still takes strips, with four waves to a strip and (the last five, from 6144 and 12288 strips on) one: two key blocks
# at a time and three, a position more than a strip and one less
STRIPS = [(1, 1, 15, 18, 128, 15, "f16"), (1, 2, 17, 31, 64, 17, "f32"), (2, 1, 9, 17, 128, 7, "f32"), (1, 1, 33, 34, 64, 31, "bf16"), (1, 1, 33, 34, 32, 31, "f32"),
          (1, 1, 63, 66, 16, 63, "f16"), (1, 1, 47, 50, 16, 47, "f32"), (32, 1, 47, 54, 128, 47, "f16"),
          (33, 1, 47, 54, 128, 47, "f16"), (33, 1, 47, 54, 128, 47, "bf16"), (71, 1, 29, 34, 128, 29, "f32"), (66, 1, 47, 54, 64, 47, "f32"), (66, 1, 49, 57, 64, 49, "f32")]


@pytest.mark.parametrize("B,heads,H,W,D,k,dtype", STRIPS)
def test_fused_forward_in_strips(oracle, B, heads, H, W, D, k, dtype):
    """Against the oracle, and, with values that are not finite, the outputs whose windows do not hold them are the same."""
    p = synth.Problem(B, heads, H, W, D, k, dtype)
    assert _fused_runs_in_strips(p)
    host = synth.make_inputs(synth.Problem(1, heads, H, W, D, k, dtype), seed=H * W + k, rpb_std=0.5)
    q, key, v = (synth.to_device(host[n], dtype).expand(B, -1, -1, -1, -1).contiguous() for n in ("q", "k", "v"))
    rpb, lse = synth.to_device(host["rpb"], dtype), torch.empty(q.shape[:4], device="cuda")
    out = na.na2d_fused_fwd(q, key, v, rpb, p.default_scale, k, torch.empty_like(q), lse)
    want, want_lse = oracle.fwd(*(host[n].astype(np.float64) for n in ("q", "k", "v", "rpb")), p.default_scale, k, return_lse=True)
    for b in {0, B - 1}:
        assert_close("out", out[b:b + 1], want, dtype)
        assert_close("lse", lse[b:b + 1], want_lse, "f32")
    v2 = v.clone()
    v2[B // 2, 0, 1, 2, 5], v2[B // 2, 0, H - 1, W - 1, 6] = float("inf"), float("nan")
    got = F.na2d(q, key, v2, rpb, kernel_size=k)
    first = lambda n: (torch.arange(n, device="cuda") - k // 2).clamp(0, n - k)
    sees = lambda y, x: ((first(H) <= y) & (y < first(H) + k))[:, None] & ((first(W) <= x) & (x < first(W) + k))[None, :]
    hit = torch.zeros_like(out, dtype=torch.bool)
    hit[B // 2, 0, :, :, 5], hit[B // 2, 0, :, :, 6] = sees(1, 2), sees(H - 1, W - 1)
    assert torch.equal(~torch.isfinite(got), hit)
    # (next to a spoilt output added up in another order: k * k independent roundings of at most 2^-25 of a sum below 1 or so, k * 2^-25 to 2^-19)
    ulp = {"f32": 2.0 ** -20, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[dtype]
    torch.testing.assert_close(got[~hit].float(), out[~hit].float(), rtol=ulp, atol=2.0 ** -19 if dtype == "f32" else ulp / 4)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])   # the types whose weights enter in two halves
@pytest.mark.parametrize("planes", [1, 33])           # four waves to a strip and one
def test_small_weights_in_strips(planes, dtype):
    """One key takes all but 2e-8 of every weight and has no value; the values of the others are large."""
    H, W, D, k = 47, 54, 128, 47
    assert _fused_runs_in_strips(synth.Problem(planes, 1, H, W, D, k, dtype))
    q, key, v = (torch.zeros(planes, 1, H, W, D, device="cuda", dtype=synth.TORCH_DTYPES[dtype]) for _ in range(3))
    rpb = torch.zeros(1, 2 * k - 1, 2 * k - 1, device="cuda", dtype=q.dtype)
    rpb[:, k - 1, k - 1] = 39 * np.log(2) - np.log(3)
    v[..., 1::2, :] = 6e4
    out = F.na2d(q, key, v, rpb, kernel_size=k)[..., 0::2, :].double()
    columns = torch.arange(W)
    first = (columns - k // 2).clamp(0, W - k)
    large = k * ((columns >= first[:, None]) & (columns < first[:, None] + k))[0::2, 1::2].sum(1).double()
    p = np.exp(-rpb[0, k - 1, k - 1].item())
    want = (large * p * v[0, 0, 0, 1, 0].item() / (1 + (k * k - 1) * p)).cuda()[None, None, None, :, None]
    # fp16: a weight, scaled by 2^15, is three times the type's smallest number but for the rounding of the table's entry (0.8 %)
    assert (out / want - 1).abs().max() < {"f16": 0.02, "bf16": 2.0 ** -7}[dtype]
