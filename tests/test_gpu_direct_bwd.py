"""The backward over 4 x 4 patches (na2d_direct_bwd) against the all-double oracle: remainders of patches, tiles and streamed rows,
each tile shape, the smallest and widest windows it takes, both counts of image buffers; what it refuses; values that are not
finite; upstream gradients of any scale."""
from __future__ import annotations

import numpy as np
import pytest
import torch

from gpu_util import Stages, assert_close, assert_close_rpb
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth

pytestmark = pytest.mark.gpu


def direct(st: Stages, with_rpb_grad=True):
    p = st.p
    prob = na.problem(p.B, p.heads, p.H, p.W, p.D, p.k, st.tdtype)
    ws = torch.empty(na.na2d_direct_bwd_workspace_bytes(prob), dtype=torch.uint8, device="cuda")
    assert ws.numel() > 0
    grads = [torch.empty_like(st.q) for _ in range(3)]
    d_rpb = torch.empty((p.heads, 2 * p.k - 1, 2 * p.k - 1), dtype=torch.float32, device="cuda") if with_rpb_grad else None
    na.na2d_direct_bwd(st.q, st.key, st.v, st.rpb, st.scale, st.lse, st.dout, p.k, *grads, d_rpb, ws)
    return (*grads, d_rpb)


def assert_close_16bit(name, got, want, dtype):
    """Bounds that follow the gradients' size.  P (dP - reference), P and dS enter the sums rounded to the storage type and the result is rounded: half a unit
    of the last place (u = 2^-11 or 2^-8 of the value) at most each, in a root mean square of 0.6 of that; the terms' errors are independent: 1.2 u of the
    gradients' rms over all.  Where few keys take most of a query's weight the terms, and their errors, are up to four times those of the others: five
    standard deviations of that, and the result's own rounding, are what one element of 10^6 may be off."""
    u, err, rms = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype], np.abs(got - want), np.sqrt((want * want).mean())
    assert np.sqrt((err * err).mean()) <= 1.2 * u * rms, (name, np.sqrt((err * err).mean()) / rms)
    assert (err <= u * np.abs(want) + 24 * u * rms).all(), (name, (err - u * np.abs(want)).max() / rms)


def check(oracle, p, seed, use_rpb=True, dout_scale=1.0, scale=None, rpb_std=0.5, f32_factor=1.0):
    host = synth.make_inputs(p, seed, rpb_std=rpb_std)
    host["dout"] = host["dout"] * dout_scale
    st = Stages(p, host, use_rpb=use_rpb, scale=scale)
    host = {n: x.astype(np.float64) for n, x in host.items()}
    host["dout"] = st.dout.double().cpu().numpy()
    st.forward_fused()
    got = direct(st)
    want = oracle.bwd(host["q"], host["k"], host["v"], host["rpb"] if use_rpb else np.zeros_like(host["rpb"]), st.scale, host["dout"], p.k)
    for n, g, o in zip(("dq", "dk", "dv"), got, want):
        # the 16-bit bound is absolute for gradients of unit scale: P dP, P and dS enter the sums rounded to the storage type, k * k of them
        # per output, at most 2^-8 (bf16) or 2^-11 (fp16) of the largest term each and their errors independent
        if p.dtype == "f32" and f32_factor != 1.0:
            err, o = np.abs(g.double().cpu().numpy() - o), np.abs(o)
            assert (err <= 1e-5 * f32_factor * np.maximum(o, np.sqrt((o * o).mean()))).all(), (n, err.max())
            continue
        assert_close(n, g.double().cpu().numpy() / dout_scale, o / dout_scale, p.dtype, abs_tol=2e-3 if p.dtype != "bf16" else 2e-2)
        if p.dtype != "f32":
            assert_close_16bit(n, g.double().cpu().numpy(), o, p.dtype)
    # dS enters exactly (to 2^-24 of the largest): what remains is the lse's spacing in the weights
    if f32_factor == 1.0:
        assert_close_rpb("d_rpb", got[3].double() / dout_scale, want[3] / dout_scale)
    for a, b in zip(direct(st), got):
        assert torch.equal(a, b)
    for a, b in zip(direct(st, with_rpb_grad=False)[:3], got):
        assert torch.equal(a, b)


# maps of one patch and less, of a remainder of one to three on either axis, and each tile shape: 8 x 16, 16 x 8 and 32 x 4 positions
@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("B,heads,H,W,D,k", [
    (70, 2, 11, 11, 32, 11), (40, 2, 13, 14, 16, 13), (33, 2, 14, 17, 32, 13), (20, 3, 31, 13, 32, 11), (32, 2, 15, 38, 32, 15), (6, 2, 22, 45, 16, 21),
    (12, 2, 34, 66, 32, 21), (22, 1, 36, 65, 64, 15)])
def test_direct_backward_all_elements(oracle, dtype, B, heads, H, W, D, k):
    check(oracle, synth.Problem(B, heads, H, W, D, k, dtype), seed=H * W + k)


# what only some types take: narrow windows of 64 channels and of fp32, 128 channels
@pytest.mark.parametrize("B,heads,H,W,D,k,dtype", [
    (3, 2, 3, 3, 64, 3, "f16"), (2, 2, 9, 5, 64, 5, "bf16"), (2, 1, 30, 37, 64, 7, "f16"), (2, 2, 19, 9, 64, 9, "bf16"), (1, 1, 13, 13, 64, 13, "f16"),
    (2, 2, 5, 6, 32, 5, "f32"), (70, 1, 10, 23, 32, 7, "f32"), (3, 2, 3, 17, 16, 3, "f32"), (2, 2, 9, 21, 16, 9, "f32"), (18, 2, 33, 34, 64, 5, "f32"),
    (60, 1, 29, 33, 128, 13, "f16"), (140, 1, 15, 50, 128, 15, "bf16"), (1, 1, 45, 47, 16, 41, "f16"), (3, 2, 34, 66, 32, 31, "bf16"), (16, 1, 33, 40, 16, 31, "f32")])
def test_direct_backward_of_some_types(oracle, B, heads, H, W, D, k, dtype):
    check(oracle, synth.Problem(B, heads, H, W, D, k, dtype), seed=H + W + k, use_rpb=(H % 2 == 1))


# dS of any scale keep the precision of the bias gradient (its integers' scale follows them); a map walked by few workgroups, so that planes of
# different bounds meet in one table
@pytest.mark.parametrize("dtype,log2_scale", [("f32", -60), ("f32", 40), ("bf16", -60), ("bf16", 60), ("f16", -6), ("f16", 8)])
def test_direct_backward_follows_the_scale_of_dout(oracle, dtype, log2_scale):
    check(oracle, synth.Problem(150, 2, 13, 13, 32, 11, dtype), seed=5, dout_scale=2.0 ** log2_scale, rpb_std=0.02)


def test_direct_backward_with_large_logits(oracle):
    # exponents far from 0: fp32 moves them to another base.  A logit of up to 256 is rounded by 2^-17 (its products, the sum, the
    # difference to the base): each weight is off by up to 4 * 2^-17 = 3e-5 of itself, delta and the normalisation with them
    check(oracle, synth.Problem(64, 2, 12, 19, 32, 11, "f32"), seed=6, scale=6.0, f32_factor=10.0)


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
@pytest.mark.parametrize("B,heads,H,W,D,k", [(72, 1, 21, 22, 32, 13), (16, 2, 17, 23, 16, 11), (6, 2, 45, 38, 32, 21)])
def test_values_with_an_offset_per_channel(oracle, dtype, B, heads, H, W, D, k):
    """dP of a window then have a large common part, which must not be left to cancel between two rounded sums."""
    p = synth.Problem(B, heads, H, W, D, k, dtype)
    host = synth.make_inputs(p, seed=k)
    host["v"] = synth.round_to(host["v"] + 10 * np.random.default_rng(k).standard_normal(D).astype(np.float32), dtype)
    st = Stages(p, host)
    st.forward_fused()
    got = direct(st)
    want = oracle.bwd(*(host[n].astype(np.float64) for n in ("q", "k", "v", "rpb")), st.scale, host["dout"].astype(np.float64), k)
    for n, g, o in zip(("dq", "dk", "dv"), got, want):
        # 16 bit: P (dP - reference), P and the result rounded, each by half a unit of the last place at most.  fp32: dP is some 10 times as large as
        # dP - delta and its sum is rounded a few times
        assert np.linalg.norm(g.double().cpu().numpy() - o) <= {"f32": 1.2e-6, "f16": 2.0 ** -11, "bf16": 2.0 ** -8}[dtype] * np.linalg.norm(o), n


@pytest.mark.parametrize("dtype,where", [("f32", "dout"), ("f32", "k"), ("bf16", "v"), ("bf16", "q"), ("f16", "dout")])
def test_values_that_are_not_finite_reach_their_windows_only(dtype, where):
    """A value that is not finite: the gradients that are not finite are those of the unfused steps, which add up each window by itself."""
    B, H, W, D, k = 40, 19, 22, 32, 15
    p = synth.Problem(B, 1, H, W, D, k, dtype)
    host = synth.make_inputs(p, seed=9)
    host[where][B // 2, 0, 2, 9, 3] = np.inf
    host[where][B // 2, 0, H - 2, W - 1, 7] = np.nan
    st = Stages(p, host)
    st.forward_fused()
    got, want = direct(st), st.backward_fused()
    for n, g, o in zip(("dq", "dk", "dv", "d_rpb"), got, want):
        assert torch.equal(torch.isfinite(g), torch.isfinite(o)), n
        f = torch.isfinite(o)
        tol = {"f32": 1e-5, "f16": 2e-2, "bf16": 1e-1}[dtype]   # (the unfused steps round logits, weights, dp and ds)
        assert (g[f] - o[f]).abs().max() <= tol * max(1.0, float(o[f].float().abs().max())), n
        rel = {"f32": 1e-6, "f16": 2.0 ** -9, "bf16": 2.0 ** -6}[dtype]   # (four roundings of the unfused steps, three of these)
        assert float((g[f].double() - o[f].double()).norm()) <= rel * float(o[f].double().norm()), n


@pytest.mark.parametrize("B,H,W,D,k,dtype", [(1, 3, 3, 64, 3, "f16"), (2, 3, 4, 64, 3, "bf16"), (1, 4, 4, 16, 3, "f32"), (1, 3, 3, 16, 3, "f32"), (3, 21, 18, 16, 11, "f16"),
                                             (2, 14, 30, 32, 13, "bf16"), (4, 13, 22, 16, 9, "f32"), (1, 30, 22, 32, 15, "f16")])
def test_bias_gradient_beside_a_query_that_is_not_finite(oracle, B, H, W, D, k, dtype):
    """The cells that the query's dS reach are NaN; in the others the rest of its patch counts as ever, also where that patch holds the
    largest dS of all (or is the only one)."""
    p = synth.Problem(B, 2, H, W, D, k, dtype)
    host = synth.make_inputs(p, seed=H + D, rpb_std=0.3)
    y, x = 1, 1
    host["dout"][..., :4, :4, :] *= 1024   # (the corner's patch: its queries reach different cells)
    st = Stages(p, host)
    st.forward_fused()
    h = {n: t.astype(np.float64) for n, t in host.items()}
    h["dout"] = st.dout.double().cpu().numpy()
    h["dout"][-1, 1, y, x] = 0   # (its dS are 0 then)
    st.dout[-1, 1, y, x, 5] = float("nan")
    got = direct(st)[3].double().cpu().numpy()
    want = oracle.bwd(h["q"], h["k"], h["v"], h["rpb"], st.scale, h["dout"], k)[3]
    first = lambda i, n: min(max(i - k // 2, 0), n - k) - i + k - 1
    reached = np.zeros(want.shape, dtype=bool)
    reached[1, first(y, H):first(y, H) + k, first(x, W):first(x, W) + k] = True
    assert np.array_equal(np.isnan(got), reached) and not reached.all()
    for head in range(2):
        assert np.abs((got - want)[head][~reached[head]]).max() <= 1e-4 * np.abs(want[head][~reached[head]]).max()


def test_refused_problems_and_arguments():
    f16, f32 = torch.float16, torch.float32
    size = lambda *a: na.na2d_direct_bwd_workspace_bytes(na.problem(*a))
    assert size(2, 2, 56, 56, 32, 7, f16) == 0        # na2d_fused_bwd has its own kernels
    assert size(2, 2, 70, 70, 32, 63, f16) == 0       # its tables and images do not fit the LDS
    assert size(64, 2, 56, 56, 128, 7, f32) == 0 and size(2, 2, 56, 56, 32, 8, f16) == 0
    assert size(2, 2, 56, 56, 32, 13, f16) > 0
    x = torch.zeros(2, 2, 14, 14, 32, dtype=f16, device="cuda")
    lse = torch.zeros(2, 2, 14, 14, device="cuda")
    grads = [torch.empty_like(x) for _ in range(3)]
    with pytest.raises(na.Na2dError) as e:
        na.na2d_direct_bwd(x, x, x, None, 1.0, lse, x, 7, *grads, None, torch.empty(1 << 24, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -8
    need = size(2, 2, 14, 14, 32, 13, f16)
    with pytest.raises(na.Na2dError) as e:
        na.na2d_direct_bwd(x, x, x, None, 1.0, lse, x, 13, *grads, None, torch.empty(need - 16, dtype=torch.uint8, device="cuda"))
    assert e.value.status == -8


def test_functional_operator_takes_it():
    p = synth.Problem(2, 2, 18, 21, 32, 13, "f16")
    host = synth.make_inputs(p, 3)
    st = Stages(p, host)
    st.forward_fused()
    want = direct(st)
    leaves = [t.detach().clone().requires_grad_() for t in (st.q, st.key, st.v, st.rpb)]
    F.na2d(*leaves, kernel_size=13).backward(st.dout)
    for leaf, w in zip(leaves, want):
        assert torch.equal(leaf.grad, w.to(leaf.dtype))
