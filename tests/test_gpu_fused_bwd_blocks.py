"""Key patches of the fused backward at the edges of their 4 x 4 blocks of queries: seen from one to four blocks of columns and of rows, from rows that
fours do not divide, in images that end with the rectangle of a tile or go on past the far border, and (k = 9) in one and two chunks of rows."""
from __future__ import annotations

import pytest

from paper_2204_07143_amd import synth
from test_gpu_parity import run_all

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("H,W,k", [
    (3, 4, 3), (4, 3, 3), (17, 18, 3), (5, 6, 5), (9, 37, 5), (37, 9, 5),
    (7, 7, 7), (8, 13, 7), (13, 8, 7), (14, 14, 7), (22, 54, 7), (54, 22, 7),   # (54: a tile whose rectangle reaches the border)
    (9, 40, 9), (11, 9, 9), (24, 23, 9), (52, 33, 9),
])
@pytest.mark.parametrize("dtype,D", [("f16", 32), ("bf16", 32), ("bf16", 16)])
def test_key_patches_at_block_edges(oracle, dtype, D, H, W, k):
    run_all(oracle, synth.Problem(3, 2, H, W, D, k, dtype), seed=H * W + k + D, rpb_std=0.5)
