"""Both sides of the rules by which a 2D problem takes the plain-ALU tiles (fp32), strips shared by four waves or strips of
one wave each, and the instances that only wide windows reach: every stage, forward and backward, against the oracle."""
from __future__ import annotations

import pytest
import torch

from paper_2204_07143_amd import binding as na
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


# The strips (planes x H x ceil(W / 16)) from which on a wave keeps one to itself, in the order of the rule: k <= 5 at
# D = 128, then the fused forward at D = 64, then its logits on rows of one strip (what has no tiles there); the fused forward to k = 9 and at D = 128; the logits at
# D >= 64; the fused forward beyond k = 9.  H is no multiple of the four strips of a workgroup; W leaves 0, 1, 2 or 15
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
