"""The patch backward with two patches to a wave (16 bit, 16 and 32 channels, from 4096 patches on where the rounds of workgroups are fewer) against the
oracle: maps whose last pair has one patch or a part of one, pairs at both borders at once, rows of blocks that only the left or the right patch
meets, each tile shape, and windows whose images are loaded between the steps."""
import numpy as np
import pytest
import torch

from gpu_util import Stages, assert_close, assert_close_rpb
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth
from test_gpu_direct_bwd import assert_close_16bit, direct

pytestmark = pytest.mark.gpu


def call(st: Stages, with_rpb_grad=True):
    """The gradients, and whether there were two patches to a wave: those keep -lse / scale of a plane's queries at the head of the workspace, one patch to a wave
    pairs of log2(e) lse and delta."""
    p = st.p
    ws = torch.empty(na.na2d_direct_bwd_workspace_bytes(na.problem(p.B, p.heads, p.H, p.W, p.D, p.k, st.tdtype)), dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(st.q) for _ in range(3)]
    d_rpb = torch.empty((p.heads, 2 * p.k - 1, 2 * p.k - 1), dtype=torch.float32, device="cuda") if with_rpb_grad else None
    na.na2d_direct_bwd(st.q, st.key, st.v, st.rpb, st.scale, st.lse, st.dout, p.k, *grads, d_rpb, ws)
    lse = st.lse[0, 0].flatten()
    return (*grads, d_rpb), torch.allclose(ws[:4 * lse.numel()].view(torch.float32) * -(st.scale or 2.0 ** -100), lse, rtol=1e-5, atol=1e-5)


def assert_close_dq(got, want, st: Stages):
    """dq is the sum of P dP k less delta times the sum of P k, P dP and P rounded to the storage type (u).  A query of which one key has nearly all the weight has these terms at full
    size, where its dS and its gradient are nearly 0: scale |dP| |k| with dP = sqrt(D) and k times a unit normal, whose product is beyond 14 in 1 of 10^6 cases.
    Over all: the bound of the other gradients."""
    u, err = {"f16": 2.0 ** -11, "bf16": 2.0 ** -8}[st.p.dtype], np.abs(got - want)
    assert np.sqrt((err * err).mean()) <= 1.2 * u * np.sqrt((want * want).mean())
    assert (err <= u * np.abs(want) + 14 * u * abs(st.scale) * st.p.D ** 0.5).all(), err.max() / u


def check(oracle, p, seed, use_rpb=True, scale=None, two=True):
    """By the bounds of test_gpu_direct_bwd.  (With a scale of 0 dq and dk are 0.)"""
    st = Stages(p, synth.make_inputs(p, seed, rpb_std=0.5), use_rpb=use_rpb, scale=scale)
    st.forward_fused()
    got, was_two = call(st)
    assert was_two == two
    host = [t.double().cpu().numpy() for t in (st.q, st.key, st.v)]
    rpb = st.rpb.double().cpu().numpy() if use_rpb else np.zeros((p.heads, 2 * p.k - 1, 2 * p.k - 1))
    want = oracle.bwd(*host, rpb, st.scale, st.dout.double().cpu().numpy(), p.k)
    assert_close_dq(got[0].double().cpu().numpy(), want[0], st)
    for n, g, o in zip(("dk", "dv"), got[1:3], want[1:3]):
        assert_close(n, g.double().cpu().numpy(), o, p.dtype, abs_tol=2e-3 if p.dtype != "bf16" else 2e-2)
        if st.scale:
            assert_close_16bit(n, g.double().cpu().numpy(), o, p.dtype)
    assert_close_rpb("d_rpb", got[3].double(), want[3])
    for again in (direct(st), direct(st, with_rpb_grad=False)):
        assert all(torch.equal(a, b) for a, b in zip(again[:3], got))


# (two: False, one patch to a wave, for fewer than 4096 patches, for 256 workgroups of two, for 8 fifths of a round against 5 on a wide map)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,H,W,D,k,two", [
    (450, 1, 11, 12, 32, 11, False), (460, 1, 11, 12, 32, 11, True), (465, 1, 11, 12, 32, 11, True), (232, 2, 11, 11, 16, 11, True), (128, 2, 14, 14, 32, 13, False),
    (150, 2, 14, 14, 32, 13, True), (90, 2, 27, 13, 32, 13, True), (40, 3, 22, 23, 16, 13, False), (54, 3, 22, 23, 16, 13, True), (30, 2, 25, 40, 32, 11, True), (76, 1, 22, 33, 16, 13, True),
    (20, 1, 53, 89, 32, 13, True), (110, 3, 16, 15, 32, 15, True), (56, 3, 18, 19, 32, 15, True), (58, 2, 30, 31, 32, 21, True), (26, 1, 41, 66, 16, 19, True)])
@pytest.mark.parametrize("use_rpb", [True, False])
def test_backward_two_patches_to_a_wave(oracle, dtype, B, heads, H, W, D, k, two, use_rpb):
    check(oracle, synth.Problem(B, heads, H, W, D, k, dtype), seed=H + W + k, use_rpb=use_rpb, two=two)


@pytest.mark.parametrize("scale", [0.0, -0.3])
def test_scales(oracle, scale):
    # the products start from -lse / scale
    check(oracle, synth.Problem(470, 1, 11, 12, 32, 11, "f16"), seed=4, scale=scale)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
def test_large_logits(oracle, dtype):
    """Logits up to 1600: an exponent is off by a few units of 2^-24 of the lse, 1e-4, with one patch to a wave and with two, whose products start from -lse / scale: rounded
    once, and the sums once more at that size, it may add 1.25 of the others' error, not 1.5 (three roundings)."""
    p = synth.Problem(128, 1, 26, 27, 32, 13, dtype)
    host = synth.make_inputs(p, 5)
    host["q"], host["k"] = host["q"] * 16, host["k"] * 16

    def results(host, B):
        st = Stages(synth.Problem(B, 1, 26, 27, 32, 13, dtype), host)
        st.forward_fused()
        return call(st)

    many, two = results(host, 128)
    assert two
    halves = [results({n: x if n == "rpb" else x[i:i + 64] for n, x in host.items()}, 64) for i in (0, 64)]
    assert not any(two for _, two in halves)
    few = [torch.cat(t) if n < 3 else t[0] + t[1] for n, t in enumerate(zip(*(g for g, _ in halves)))]
    host = {n: x.astype(np.float64) for n, x in host.items()}
    want = oracle.bwd(host["q"], host["k"], host["v"], host["rpb"], p.default_scale, host["dout"], p.k)
    for n, a, b, o in zip(("dq", "dk", "dv", "d_rpb"), many, few, want):
        err = [np.sqrt(((x.double().cpu().numpy() - o) ** 2).mean()) for x in (a, b)]
        assert err[0] <= 1.25 * err[1], (n, err)


@pytest.mark.parametrize("where", ["q", "k", "v", "dout"])
@pytest.mark.parametrize("value", [float("nan"), float("inf"), 3e38])
def test_not_finite(where, value):
    """The same planes, alone (one patch to a wave) and among many (two): the same elements are finite.  3e38: finite itself, its products are not."""
    g = torch.Generator(device="cuda").manual_seed(3)
    one = {n: torch.randn((1, 1, 26, 27, 32), generator=g, device="cuda").bfloat16() for n in ("q", "k", "v", "dout")}
    one[where][0, 0, 12, 5, 7] = value
    rpb = torch.zeros((1, 25, 25), device="cuda").bfloat16()

    def grads(B):
        q, k, v, r = (t.expand(B, *t.shape[1:]).clone().requires_grad_() if t.dim() == 5 else t.clone().requires_grad_()
                      for t in (one["q"], one["k"], one["v"], rpb))
        return torch.autograd.grad(F.na2d(q, k, v, r, kernel_size=13), (q, k, v, r), one["dout"].expand(B, -1, -1, -1, -1).contiguous())

    few, many = grads(1), grads(128)
    for a, b in zip(few[:3], many[:3]):
        assert torch.equal(a[0].isfinite(), b[0].isfinite())
        f = a[0].isfinite()
        assert torch.allclose(a[0][f], b[0][f], rtol=2.0 ** -6, atol=3e-2)   # (added up in another order: two roundings of the weights to 8 bits)
    assert torch.equal(few[3].isfinite(), many[3].isfinite())
