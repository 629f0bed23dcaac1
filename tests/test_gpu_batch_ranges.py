"""Calls with more (tile position, head) units than fit the chip at once, or nearly: the batch is cut into ranges so that few places stay
empty.  An item's results are those of a call of its own, whatever range it is in; the bias gradient is the sum over the items."""
import pytest
import torch

from gpu_util import Stages, assert_close_rpb
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import synth

pytestmark = pytest.mark.gpu


def item(host, i):
    return {n: x if n == "rpb" else x[i:i + 1] for n, x in host.items()}


# ranges: of the batch, for every (tile of 16 x 8, head) unit: 264, 320, 288, 180, 520, 288, 288, 264 units in ranges of two lengths; 288 of 4 items in one
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,H,W,D,k,ranges", [
    (11, 264, 8, 16, 32, 7, 3), (11, 320, 8, 13, 32, 5, 3), (11, 72, 15, 30, 32, 7, 3), (33, 90, 9, 16, 16, 3, 4), (13, 520, 7, 7, 32, 7, 2), (11, 144, 12, 16, 32, 9, 3),
    (11, 144, 16, 13, 32, 13, 3), (11, 264, 8, 16, 64, 7, 3), (4, 288, 8, 16, 32, 7, 1),
    # (columns of key tiles: 300 and 270 of 8 tiles, in two segments)
    (10, 30, 64, 16, 32, 7, 2), (9, 15, 61, 27, 16, 3, 2),
    # (the tile kernel of grad-v and grad-k: k = 9, and a map that the ring refuses)
    (10, 72, 24, 17, 32, 9, 1), (11, 36, 100, 16, 32, 7, 1)])
def test_items_of_a_range(dtype, B, heads, H, W, D, k, ranges):
    p = synth.Problem(B, heads, H, W, D, k, dtype)
    prob = na.problem(B, heads, H, W, D, k, synth.TORCH_DTYPES[dtype])
    if na.na2d_fused_bwd_is_fused(prob):   # (the fused backward's workspace: two words a query, a partial bias gradient of each workgroup)
        up = lambda n: (n + 255) // 256 * 256
        tiles, row = -(-W // 16) * -(-H // 8) * heads, 4 * (((2 * k - 1) ** 2 + 3) // 4 * 4)
        assert na.na2d_workspace_bytes(prob, na.WS_FUSED_BWD) == 2 * up(B * heads * H * W * 4) + up(tiles * ranges * row)
    host = synth.make_inputs(p, seed=H + W + k, rpb_std=0.5)
    names = ("logits", "attn", "out", "out_fused", "lse", "dp", "ds", "dv", "dq", "dk")

    def results(p, host):
        st = Stages(p, host)
        st.forward_unfused(), st.forward_fused(), st.backward_unfused()
        fused = st.backward_fused() if k <= 9 and D <= 32 else ()
        composed = st.backward_composed() if D <= 32 else ()   # (the strips' sums at 64 channels look at the call's size)
        return [getattr(st, n) for n in names if D <= 32 or n not in ("dv", "dk")] + [*fused[:3], *composed[:3]], [st.d_rpb, *fused[3:], *composed[3:4]]

    whole, sums = results(p, host)
    parts = [torch.zeros_like(s, dtype=torch.float64) for s in sums]
    for i in range(B):
        one, s = results(synth.Problem(1, heads, H, W, D, k, dtype), item(host, i))
        for n, (a, b) in enumerate(zip(whole, one)):
            assert torch.equal(a[i:i + 1], b), f"item {i}, result {n}"
        for t, x in zip(parts, s):
            t += x
    for t, x in zip(parts, sums):
        assert_close_rpb("d_rpb", x.double(), t.cpu().numpy())
