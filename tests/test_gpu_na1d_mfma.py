"""The 16-bit 1D kernels on the matrix cores against the fp64 1D oracle: each number of key blocks at both ends of its range of
windows, sequences that end inside a group of 16 queries, inside a wave and inside a tile, calls of few and of many tiles, and
values that are not finite."""
import numpy as np
import pytest
import torch

from oracle import na1d_oracle as o1
from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import synth

from gpu_util import assert_close, assert_close_rpb, to_np

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


def backward(p, seed, use_rpb=True, rpb_std=0.02, dout_scale=1.0, edit=None):
    host = synth.make_inputs_1d(p, seed, rpb_std=rpb_std)
    host["dout"] = host["dout"] * dout_scale
    if edit:
        edit(host)
    q, key, v, dout = (synth.to_device(host[n], p.dtype) for n in ("q", "k", "v", "dout"))
    rpb = synth.to_device(host["rpb"], p.dtype) if use_rpb else None
    lse = torch.empty(q.shape[:3], dtype=torch.float32, device="cuda")
    na.na1d_fused_fwd(q, key, v, rpb, p.default_scale, p.k, torch.empty_like(q), lse)
    ws = torch.empty(na.na1d_fused_bwd_workspace_bytes(na.problem_1d(p.B, p.heads, p.L, p.D, p.k, q.dtype)), dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(q) for _ in range(3)] + [torch.empty((p.heads, 2 * p.k - 1), dtype=torch.float32, device="cuda")]
    na.na1d_fused_bwd(q, key, v, rpb, p.default_scale, lse, dout, p.k, *grads, ws)
    h = [t.double().cpu().numpy() for t in (q, key, v)]
    table = rpb.double().cpu().numpy() if use_rpb else np.zeros((p.heads, 2 * p.k - 1))
    with np.errstate(all="ignore"):
        return grads, o1.bwd(*h, table, p.default_scale, dout.double().cpu().numpy(), p.k)


# (the last two: 512 tiles and more, four groups of queries to a wave of the forward)
SIZES = [(B, heads, L, k) for B, heads, L, ks in [
    (2, 2, 63, (3, 17, 19, 33, 35, 49, 51, 63)), (1, 3, 65, (3, 17, 19, 33, 35, 49, 51, 63)), (1, 2, 193, (7, 31, 63)), (2, 1, 1025, (17, 35, 63)),
    (130, 4, 67, (3, 17, 19, 33, 35, 49, 51, 63)), (90, 2, 531, (3, 33, 63))] for k in ks]


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,L,k", SIZES)
def test_forward_blocks(dtype, B, heads, L, k):
    out, lse, (want, want_lse) = forward(synth.Problem1D(B, heads, L, 32, k, dtype), seed=L + k, use_rpb=L % 2 == 1 and L != 65, rpb_std=0.5)
    assert_close("out", out, want, dtype)
    assert_close("lse", lse, want_lse, "f32")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,L,k", SIZES)
def test_backward_blocks(dtype, B, heads, L, k):
    got, want = backward(synth.Problem1D(B, heads, L, 32, k, dtype), seed=L + k, use_rpb=L % 2 == 1 and L != 65, rpb_std=0.5)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        assert_close(n, x, y, dtype)
    assert_close_rpb("d_rpb", got[3], want[3])


@pytest.mark.parametrize("dtype,log2_scale", [("f16", -6), ("f16", 8), ("bf16", -15), ("bf16", 10)])
def test_backward_follows_the_scale_of_dout(dtype, log2_scale):
    """(fp16: dout far from its subnormals; the bias gradient's integers count 2^-42)"""
    s = 2.0 ** log2_scale
    got, want = backward(synth.Problem1D(3, 2, 300, 32, 21, dtype), seed=3, dout_scale=s)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        assert_close(n, x.double() / s, y / s, dtype)
    assert_close_rpb("d_rpb", got[3].double() / s, want[3] / s)


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("what", ["q", "k", "v", "dout"])
def test_backward_not_finite_stays_in_its_windows(dtype, what):
    def edit(host):
        host[what][0, 0, 60, 3] = np.nan
        host[what][0, 1, 0, 5] = np.nan

    k, L = 7, 200
    got, want = backward(synth.Problem1D(1, 2, L, 32, k, dtype), seed=9, edit=edit)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        x = to_np(x)
        assert np.isfinite(y).all() == (n == "dv" and what == "v") and np.array_equal(np.isfinite(x), np.isfinite(y)), n
        zero = lambda t: np.where(np.isfinite(y), t, 0.0)
        assert_close(n, zero(x), zero(y), dtype)


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


@pytest.mark.parametrize("dtype", ["f32", "f16", "bf16"])
def test_forward_with_masked_bias_cells(dtype):
    """Windows whose first keys are masked by a bias of -inf, alone and next to values that are not finite just outside of them."""
    k, L = 7, 200

    def edit(host):
        host["rpb"][:, : k // 2 + 2] = -np.inf   # (the first keys, and at the right end those that come first there)
        host["v"][0, 0, 60, 3] = np.nan
        host["k"][0, 1, 100, 5] = np.inf

    with np.errstate(all="ignore"):
        out, lse, (want, want_lse) = forward(synth.Problem1D(1, 2, L, 32, k, dtype), seed=9, edit=edit)
    got, finite = to_np(out), np.isfinite(want)
    assert not finite.all() and finite.mean() > 0.9 and np.array_equal(np.isfinite(got), finite)
    assert_close("out", np.where(finite, got, 0.0), np.where(finite, want, 0.0), dtype)
    finite = np.isfinite(want_lse)
    assert np.array_equal(np.isfinite(to_np(lse)), finite)
    assert_close("lse", np.where(finite, to_np(lse), 0.0), np.where(finite, want_lse, 0.0), "f32")


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("k", [7, 31, 63])
def test_bias_gradient_of_large_terms_that_cancel(dtype, k):
    """Queries 16 positions apart that see the same keys' values: the first sixteen's dS are large, the third's the same with the other sign, and what is
    left of a cell is the second's, which an fp32 sum of the three would have lost."""
    def edit(host):
        for n in ("v", "dout"):
            host[n][:] = np.sign(host[n])   # (their products are whole numbers: the same with either sign)
        for n in ("q", "k", "v"):
            host[n][:] = np.tile(host[n][:, :, :16], (1, 1, 32, 1))
        dout = host["dout"][:, :, 64:80].copy()
        small = host["dout"][:, :, 80:96].copy()
        host["dout"][:] = 0
        host["dout"][:, :, 64:80], host["dout"][:, :, 80:96], host["dout"][:, :, 96:112] = 2.0 ** 11 * dout, 2.0 ** -9 * small, -2.0 ** 11 * dout

    got, want = backward(synth.Problem1D(1, 2, 512, 32, k, dtype), seed=k, edit=edit)
    assert_close_rpb("d_rpb", got[3], want[3])


def test_a_value_that_is_not_finite_costs_no_multiple_of_a_pass():
    """One infinite key per plane: the results around it are worked out once more by a few waves, which the call waits for (kernels alone, out of a graph)."""
    B, heads, L, k = 64, 2, 3136, 31
    g = torch.Generator(device="cuda").manual_seed(1)
    q, key, v, dout = (torch.randn((B, heads, L, 32), generator=g, device="cuda").half() for _ in range(4))
    ws = torch.empty(na.na1d_fused_bwd_workspace_bytes(na.problem_1d(B, heads, L, 32, k, q.dtype)), dtype=torch.uint8, device="cuda")
    out, grads, lse = torch.empty_like(q), [torch.empty_like(q) for _ in range(3)], torch.empty(B, heads, L, device="cuda")
    d_rpb = torch.empty(heads, 2 * k - 1, device="cuda")

    def call():
        na.na1d_fused_fwd(q, key, v, None, 0.18, k, out, lse)
        na.na1d_fused_bwd(q, key, v, None, 0.18, lse, dout, k, *grads, d_rpb, ws)

    def best():
        call()
        torch.cuda.synchronize()
        graph, times = torch.cuda.CUDAGraph(), []
        with torch.cuda.graph(graph):
            for _ in range(10):
                call()
        for _ in range(6):
            a, b = (torch.cuda.Event(enable_timing=True) for _ in range(2))
            a.record()
            graph.replay()
            b.record()
            b.synchronize()
            times.append(a.elapsed_time(b))
        return min(times)

    finite = best()
    key[:, :, L // 2, 3] = float("inf")
    assert best() <= 2.5 * finite   # (1.9; with the vectors read from memory, one position at a time, 3.1)
