"""The 1D backward in one kernel (16 bit, k <= 17) against the fp64 1D oracle: sequences that end on either side of a tile of 224 positions, of its
neighbours' 16, and of the last keys' longer reach; values that are not finite on both sides of a tile's border."""
import numpy as np
import pytest

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
