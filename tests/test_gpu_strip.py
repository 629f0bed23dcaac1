"""The strip kernels (na2d_strip.hip) where they can go wrong: maps of one strip, a strip and a remainder, a strip more
than the windows' reach; and values that are not finite, which must reach exactly the outputs whose window holds them."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth
from gpu_util import assert_close

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("H,W,D,k", [(15, 16, 32, 15), (17, 33, 16, 17), (19, 19, 64, 19), (34, 49, 32, 33), (63, 65, 16, 63), (13, 31, 128, 13)])
def test_forward_at_strip_edges(oracle, H, W, D, k, dtype):
    p = synth.Problem(1, 2, H, W, D, k, dtype)
    host = synth.make_inputs(p, seed=H * W + D)
    q, key, v, rpb = (synth.to_device(host[n], dtype) for n in ("q", "k", "v", "rpb"))
    out = F.na2d(q, key, v, rpb, kernel_size=k)
    h = {n: host[n].astype(np.float64) for n in host}
    assert_close("out", out, oracle.fwd(h["q"], h["k"], h["v"], h["rpb"], p.default_scale, k), dtype)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])            # the types whose weights enter in two halves
@pytest.mark.parametrize("planes", [1, 100])   # (over patches, shared by waves and not; in strips: test_gpu_routes.py)
def test_small_weights_of_large_values(oracle, planes, dtype):
    # One key takes all but 2.5e-8 of every weight and the values next to it are large: where a query's own column holds
    # zeros its output is the sum of some 480 weights below 2^-25 times 6e4 (about 0.7).  The logits are the bias alone.
    H, W, D, k = 62, 31, 16, 31
    p = synth.Problem(planes, 1, H, W, D, k, dtype)
    host = synth.make_inputs(synth.Problem(1, 1, H, W, D, k, dtype), seed=8)
    host["q"][:] = 0
    host["rpb"][:] = 0
    host["rpb"][:, k - 1, k - 1] = 17.5
    host["v"][..., 0::2, :] = 0
    host["v"][..., 1::2, :] = synth.round_to(np.full(D, 6e4, dtype=np.float32), dtype)
    q, key, v, rpb = (synth.to_device(host[n], dtype) for n in ("q", "k", "v", "rpb"))
    q, key, v = (t.expand(p.B, -1, -1, -1, -1).contiguous() for t in (q, key, v))
    out = F.na2d(q, key, v, rpb, kernel_size=k)
    want = oracle.fwd(*(host[n].astype(np.float64) for n in ("q", "k", "v", "rpb")), p.default_scale, k)
    for b in {0, planes - 1}:
        # columns whose own value is zero (the others are 6e4 themselves)
        assert_close("out", out[b:b + 1, :, :, 0::2], want[:, :, :, 0::2], dtype)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("H,W,k", [(15, 17, 15), (19, 21, 17), (33, 22, 21), (63, 63, 63)])
def test_logits_whose_rows_are_shared_by_workgroups(oracle, H, W, k, dtype):
    # One plane alone (every window row of a strip in a wave of its own) and many planes (all of a strip's rows in one
    # workgroup) write the same bits, and the oracle's.
    planes = 1 + 2048 // (H * ((W + 15) // 16)) if k < 63 else 20
    p = synth.Problem(planes, 1, H, W, 16, k, dtype)
    host = synth.make_inputs(synth.Problem(1, 1, H, W, 16, k, dtype), seed=k)
    q, key, rpb = (synth.to_device(host[n], dtype) for n in ("q", "k", "rpb"))
    empty = lambda b: torch.full((b, 1, H, W, k * k), float("nan"), dtype=q.dtype, device="cuda")
    one = na.na2d_qk_rpb(q, key, rpb, p.default_scale, k, empty(1))
    assert_close("logits", one, oracle.qk_rpb(*(host[n].astype(np.float64) for n in ("q", "k", "rpb")), p.default_scale, k), dtype)
    many = na.na2d_qk_rpb(*(t.expand(planes, -1, -1, -1, -1).contiguous() for t in (q, key)), rpb, p.default_scale, k, empty(planes))
    assert all(torch.equal(many[b:b + 1], one) for b in (0, planes // 2, planes - 1))


def test_bias_entries_do_not_wait_for_each_other():
    # one entry at a time behind each store's condition made logits with a bias take 1.5 times as long as without
    torch.manual_seed(5)
    B, H, W, D, k = 2, 100, 134, 16, 45
    q, key = (torch.randn(B, 1, H, W, D, device="cuda") for _ in range(2))
    rpb = torch.randn(1, 2 * k - 1, 2 * k - 1, device="cuda")
    out = torch.empty(B, 1, H, W, k * k, device="cuda")

    def best(bias):
        times = []
        for _ in range(8):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                na.na2d_qk_rpb(q, key, bias, 0.25, k, out)
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    assert best(rpb) <= 1.25 * best(None)   # (1.01 to 1.07 now)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_infinities_reach_their_windows_only(dtype):
    H, W, D, k, y, x = 21, 40, 32, 15, 2, 20
    torch.manual_seed(1)
    dt = synth.TORCH_DTYPES[dtype]
    q, key, v, dout = (torch.randn(1, 1, H, W, D, device="cuda").to(dt) for _ in range(4))
    want = F.na2d(q, key, v, None, kernel_size=k)
    v2 = v.clone()
    v2[0, 0, y, x, 5] = float("inf")
    got = F.na2d(q, key, v2, None, kernel_size=k)
    attn = F.na2d_softmax(F.na2d_qk_rpb(q, key, None, k), q, k)
    got_av = F.na2d_av(attn, v2, k)
    first = lambda n, L: (torch.arange(n, device="cuda") - k // 2).clamp(0, L - k)
    sees = lambda c, L: (first(L, L) <= c) & (c < first(L, L) + k)
    hit = sees(y, H)[:, None] & sees(x, W)[None, :]
    for g in (got, got_av):
        assert torch.equal(torch.isinf(g[0, 0, :, :, 5]) | torch.isnan(g[0, 0, :, :, 5]), hit)
        rest = torch.ones(D, dtype=torch.bool, device="cuda")
        rest[5] = False
        assert torch.isfinite(g[..., rest]).all()
    assert (got[0, 0, :, :, 5][~hit].float() - want[0, 0, :, :, 5][~hit].float()).abs().max() < 8e-3
    # grad-v: the same for an upstream gradient that is not finite, seen by the keys of that query's window
    dout[0, 0, y, x, 5] = float("inf")
    leaf = v.clone().requires_grad_()
    F.na2d_av(attn, leaf, k).backward(dout)
    sy, sx = max(0, min(y - k // 2, H - k)), max(0, min(x - k // 2, W - k))
    want_hit = torch.zeros(H, W, dtype=torch.bool, device="cuda")
    want_hit[sy:sy + k, sx:sx + k] = True
    assert torch.equal(~torch.isfinite(leaf.grad[0, 0, :, :, 5]), want_hit)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("planes,H,W,D,k", [(1, 17, 33, 16, 15), (370, 17, 17, 16, 15), (1, 21, 40, 32, 21), (1, 13, 18, 128, 13), (420, 15, 17, 128, 15)])
def test_values_that_are_not_finite_change_no_other_output(planes, H, W, D, k, dtype):
    # (the weighted sum in strips: four, two and one positions side by side in a wave; the fused forward over patches, in strips: test_gpu_routes.py)
    torch.manual_seed(3)
    q, key, v = (torch.randn(planes, 1, H, W, D, device="cuda").to(synth.TORCH_DTYPES[dtype]) for _ in range(3))
    attn = F.na2d_softmax(F.na2d_qk_rpb(q, key, None, k), q, k)
    b, spots = planes // 2, [(2, 1, 5, float("inf")), (H - 3, W - 2, 5, -float("inf")), (H // 2, 0, 9, float("nan"))]
    v2 = v.clone()
    for y, x, d, value in spots:
        v2[b, 0, y, x, d] = value
    first = lambda n, L: (torch.arange(n, device="cuda") - k // 2).clamp(0, L - k)
    sees = lambda c, L: (first(L, L) <= c) & (c < first(L, L) + k)
    for op in (lambda t: F.na2d(q, key, t, None, kernel_size=k), lambda t: F.na2d_av(attn, t, k)):
        want, got = op(v).float(), op(v2).float()
        for y, x, d, value in spots:
            hit = sees(y, H)[:, None] & sees(x, W)[None, :]
            want[b, 0, :, :, d][hit] += value   # (an infinity of each sign: NaN)
        # one rounding to the storage type (outputs next to a spoilt one are added up in another order)
        ulp = {"f32": 2.0 ** -20, "f16": 2.0 ** -10, "bf16": 2.0 ** -7}[dtype]
        torch.testing.assert_close(got, want, rtol=ulp, atol=ulp / 4, equal_nan=True)


@pytest.mark.parametrize("B,H,W,D,k,dtype", [(8, 64, 64, 32, 21, "bf16"), (4, 56, 56, 128, 9, "f16"), (8, 56, 56, 64, 9, "f32")])
def test_tensors_of_nan_take_no_multiple_of_the_time(B, H, W, D, k, dtype):
    # a step that diverged: each output is worked out once more from its own window, and that must not go the long way
    torch.manual_seed(4)
    q, key, v = (torch.randn(B, 1, H, W, D, device="cuda").to(synth.TORCH_DTYPES[dtype]) for _ in range(3))
    attn = F.na2d_softmax(F.na2d_qk_rpb(q, key, None, k), q, k)
    out, nan = torch.empty_like(q), torch.full_like(v, float("nan"))

    def best(call):
        times = []
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            for _ in range(5):
                call()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    fused = lambda t: best(lambda: na.na2d_fused_fwd(q, key, t, None, D ** -0.5, k, out))
    finite = fused(v)
    assert fused(nan) <= 10 * finite and torch.isnan(out).all()   # (D logits of every slot where one would do: 30 to 120 times)
    for op in (na.na2d_av, na.na2d_av_bwd_v):
        finite = best(lambda: op(attn, v, k, out))
        assert best(lambda: op(attn, nan, k, out)) <= 3 * finite and torch.isnan(out).all()   # (10 times with the whole window)
