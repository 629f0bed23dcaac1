"""The rule by which a 2D fp32 problem takes the plain-ALU tiles or the strips: every stage on both sides of it, against the oracle."""
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
