"""The 16-bit 1D kernels on the matrix cores against the fp64 1D oracle: each number of key blocks at both ends of its range of
windows, sequences that end inside a group of 16 queries, inside a wave and inside a tile, calls of few and of many tiles, and
values that are not finite."""
import numpy as np
import pytest
import torch

from oracle import na1d_oracle as o1
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import synth

from gpu_util import assert_close, to_np

pytestmark = pytest.mark.gpu


def forward(p, seed, use_rpb=True, rpb_std=0.02, edit=None):
    host = synth.make_inputs_1d(p, seed, rpb_std=rpb_std)
    if edit:
        edit(host)
    q, key, v = (synth.to_device(host[n], p.dtype) for n in ("q", "k", "v"))
    rpb = synth.to_device(host["rpb"], p.dtype) if use_rpb else None
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    na.na1d_fused_fwd(q, key, v, rpb, p.default_scale, p.k, out, lse)
    h = [t.double().cpu().numpy() for t in (q, key, v)] + [rpb.double().cpu().numpy() if use_rpb else None]
    return out, lse, o1.fwd(*h, p.default_scale, p.k, return_lse=True)


# (the last two: 512 tiles and more, four groups of queries to a wave)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,L,k", [(B, heads, L, k) for B, heads, L, ks in [
    (2, 2, 63, (3, 17, 19, 33, 35, 49, 51, 63)), (1, 3, 65, (3, 17, 19, 33, 35, 49, 51, 63)), (1, 2, 193, (7, 31, 63)), (2, 1, 1025, (17, 35, 63)),
    (130, 4, 67, (3, 17, 19, 33, 35, 49, 51, 63)), (90, 2, 531, (3, 33, 63))] for k in ks])
def test_forward_blocks(dtype, B, heads, L, k):
    out, lse, (want, want_lse) = forward(synth.Problem1D(B, heads, L, 32, k, dtype), seed=L + k, use_rpb=L % 2 == 1 and L != 65, rpb_std=0.5)
    assert_close("out", out, want, dtype)
    assert_close("lse", lse, want_lse, "f32")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("what", ["q", "k", "v"])
def test_forward_not_finite_stays_in_its_windows(dtype, what):
    """(a key whose product with a query is -inf leaves that query finite)"""
    k, L, at = 7, 200, 60

    def edit(host):
        host[what][0, 0, at, 3] = np.inf
        host[what][0, 1, 0, 5] = np.nan

    with np.errstate(all="ignore"):
        out, _, (want, _) = forward(synth.Problem1D(1, 2, L, 32, k, dtype), seed=9, edit=edit)
    got = to_np(out)
    assert not np.isfinite(want).all() and np.array_equal(np.isfinite(got), np.isfinite(want))
    zero = lambda x: np.where(np.isfinite(want), x, 0.0)
    assert_close("out", zero(got), zero(want), dtype)
