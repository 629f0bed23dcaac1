"""The 1D backward in one kernel (16 bit, k <= 17) against the fp64 1D oracle: sequences that end on either side of a tile of 224 positions, of its
neighbours' 16, and of the last keys' longer reach; values that are not finite on both sides of a tile's border.  And the calls that two kernels serve."""
import numpy as np
import pytest
import torch

from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import synth

from gpu_util import assert_close, assert_close_rpb, to_np
from test_gpu_na1d_mfma import backward

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("L", [17, 207, 224, 225, 232, 240, 241, 447, 448, 464, 465])
@pytest.mark.parametrize("k", [3, 11, 17])
def test_tiles(dtype, L, k):
    got, want = backward(synth.Problem1D(2, 3, L, 32, k, dtype), seed=L + k, use_rpb=L % 3 != 0, rpb_std=0.5)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        assert_close(n, x, y, dtype)
    assert_close_rpb("d_rpb", got[3], want[3])


@pytest.mark.parametrize("what", ["q", "k", "v", "dout"])
@pytest.mark.parametrize("at", [208, 223, 224, 231])
def test_not_finite_beside_a_border(what, at):
    def edit(host):
        host[what][0, 0, at, 3] = np.nan

    got, want = backward(synth.Problem1D(1, 1, 460, 32, 17, "bf16"), seed=at, edit=edit)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        assert np.array_equal(np.isfinite(to_np(x)), np.isfinite(y)), n
        zero = lambda t: np.where(np.isfinite(y), t, 0.0)
        assert_close(n, zero(to_np(x)), zero(y), "bf16")


def call(q, k, v, dout, rpb, kernel_size):
    """The gradients, and whether two kernels made them: they keep every query's delta = <dout, out> at the head of the workspace, where the one kernel has its tables."""
    planes, scale, n = q.shape[:2], q.shape[3] ** -0.5, q.shape[0] * q.shape[1] * q.shape[2]
    out, lse = torch.empty_like(q), torch.empty(q.shape[:3], device="cuda")
    na.na1d_fused_fwd(q, k, v, rpb, scale, kernel_size, out, lse)
    ws = torch.zeros(na.na1d_fused_bwd_workspace_bytes(na.problem_1d(*planes, q.shape[2], q.shape[3], kernel_size, q.dtype)), dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(q) for _ in range(3)] + [torch.empty((q.shape[1], 2 * kernel_size - 1), device="cuda")]
    na.na1d_fused_bwd(q, k, v, rpb, scale, lse, dout, kernel_size, *grads, ws)
    delta = (dout.float() * out.float()).sum(-1).flatten()
    return grads, torch.allclose(ws[:4 * n].view(torch.float32), delta, atol=0.05)


# (260 sequences of 225 to 256 and 110 of 1000: one tile of 256 instead of two of 224, four instead of five; 1700 of 250)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,L,k", [(130, 2, 225, 17), (130, 2, 241, 3), (130, 2, 256, 11), (55, 2, 1000, 7), (850, 2, 250, 7)])
def test_two_kernels(dtype, B, heads, L, k):
    """Calls whose tiles of 224 would take a round of workgroups more: the oracle's results, and of an item the bits that it has in a call of its own, which is
    one kernel's."""
    p = synth.Problem1D(B, heads, L, 32, k, dtype)
    host = synth.make_inputs_1d(p, seed=L + k, rpb_std=0.5)
    q, key, v, dout, rpb = (synth.to_device(host[n], dtype) for n in ("q", "k", "v", "dout", "rpb"))
    grads, two = call(q, key, v, dout, rpb, k)
    assert two
    for i in (0, B // 2, B - 1):
        one, two = call(*(t[i:i + 1].contiguous() for t in (q, key, v, dout)), rpb, k)
        assert not two and all(torch.equal(a[i:i + 1], b) for a, b in zip(grads[:3], one))
    got, want = backward(p, seed=L + k, rpb_std=0.5)
    for n, x, y in zip(("dq", "dk", "dv"), got, want):
        assert_close(n, x, y, dtype)
    assert_close_rpb("d_rpb", got[3], want[3])


@pytest.mark.parametrize("B,heads,L", [(128, 2, 256), (128, 2, 250), (130, 4, 200), (64, 2, 1792), (64, 10, 490)])
def test_one_kernel(B, heads, L):
    """On the other side of the rule's limits: 512 workgroups, as many tiles of 224 as of 256, more tiles of 256 than one round holds."""
    g = torch.Generator(device="cuda").manual_seed(L)
    q, k, v, dout = (torch.randn((B, heads, L, 32), generator=g, device="cuda").half() for _ in range(4))
    assert not call(q, k, v, dout, torch.zeros((heads, 13), device="cuda").half(), 7)[1]
