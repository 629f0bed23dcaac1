"""Key side of the patch backward with two waves per patch (16 bit, k > 13, few patches) against the oracle on both sides of the rule, with
and without a bias and its gradient: maps of one patch row, remainders of patches, of tiles and of the eight rows of a step; a value that
is not finite reaches what the single waves let it reach."""
import pytest
import torch

from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth
from test_gpu_direct_bwd import check

pytestmark = pytest.mark.gpu


# (patches: 16 .. 2048 take pairs, 2080 and more do not)
@pytest.mark.parametrize("dtype", ["f16", "bf16"])
@pytest.mark.parametrize("B,heads,H,W,D,k", [
    (1, 1, 15, 15, 32, 15), (2, 3, 21, 22, 16, 21), (4, 2, 17, 50, 64, 15), (3, 1, 41, 37, 32, 19), (8, 2, 45, 43, 32, 21), (5, 4, 39, 41, 16, 17),
    (5, 4, 40, 44, 32, 15),
    (1, 2, 131, 18, 32, 17), (1, 1, 203, 27, 16, 15), (8, 1, 76, 21, 64, 19)])   # (maps of many tile rows)
@pytest.mark.parametrize("use_rpb", [True, False])
def test_backward_in_pairs(oracle, dtype, B, heads, H, W, D, k, use_rpb):
    check(oracle, synth.Problem(B, heads, H, W, D, k, dtype), seed=H + W + k, use_rpb=use_rpb)


@pytest.mark.parametrize("where", ["q", "k", "dout"])
def test_not_finite_in_pairs(where):
    """The same planes, alone (pairs) and among many (one wave per patch): the same elements are finite."""
    g = torch.Generator(device="cuda").manual_seed(3)
    one = {n: torch.randn((1, 1, 26, 27, 32), generator=g, device="cuda").half() for n in ("q", "k", "v", "dout")}
    one[where][0, 0, 12, 5, 7] = float("nan")
    rpb = torch.zeros((1, 29, 29), device="cuda").half()

    def grads(B):
        q, k, v, r = (t.expand(B, *t.shape[1:]).clone().requires_grad_() if t.dim() == 5 else t.clone().requires_grad_()
                      for t in (one["q"], one["k"], one["v"], rpb))
        return torch.autograd.grad(F.na2d(q, k, v, r, kernel_size=15), (q, k, v, r), one["dout"].expand(B, -1, -1, -1, -1).contiguous())

    few, many = grads(1), grads(60)
    for a, b in zip(few[:3], many[:3]):
        assert torch.equal(a[0].isfinite(), b[0].isfinite()) and not a.isfinite().all()
        assert torch.allclose(a[0].nan_to_num(0), b[0].nan_to_num(0), rtol=0, atol=4e-3)
    assert torch.equal(few[3].isfinite(), many[3].isfinite())
