"""The library under HIP graph capture: every entry point only launches kernels on the stream it is given
(no allocation, no synchronisation, no memset or copy), so a captured sequence must replay to the bits of
the eager calls, on every replay, with eager work and synchronisations of the program in between."""
import pytest
import torch

from paper_2204_07143_amd import binding as na
from paper_2204_07143_amd import functional as F
from paper_2204_07143_amd import synth

from gpu_util import Stages

pytestmark = pytest.mark.gpu


def _run_everything(st: Stages):
    st.forward_unfused()
    st.forward_fused()
    st.backward_unfused()
    c = st.backward_composed()
    f = st.backward_fused()
    return [st.logits, st.attn, st.out, st.out_fused, st.lse, st.dp, st.dv, st.ds, st.dq, st.dk, st.d_rpb, *c[:4], *f]


@pytest.mark.parametrize("k,dtype", [(7, "f16"), (5, "bf16"), (9, "f16"), (3, "f32")])
def test_graph_replays_match_eager(k, dtype):
    p = synth.Problem(5, 2, 27, 41, 32, k, dtype)
    host = synth.make_inputs(p, seed=60 + k)
    st = Stages(p, host)
    eager = [t.clone() for t in _run_everything(st)]   # also the warm-up: code objects loaded, LDS limits set
    torch.cuda.synchronize()

    # the captured calls write into buffers that live as long as the graph
    class Holder(Stages):
        pass
    gst = Holder(p, host)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = _run_everything(gst)
    for replay in range(4):
        for t in outs:
            t.fill_(float("nan")) if t.is_floating_point() else t.zero_()
        # eager work of the program between the replays, on the same stream, and a synchronisation
        other = _run_everything(st)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i, (a, b) in enumerate(zip(outs, eager)):
            assert torch.equal(a, b), f"replay {replay}: output {i} differs from the eager result"
        for i, (a, b) in enumerate(zip(other, eager)):
            assert torch.equal(a, b), f"replay {replay}: eager output {i} changed"


def test_noalloc_entry_point_under_capture():
    p = synth.Problem(4, 2, 20, 33, 32, 7, "f16")
    host = synth.make_inputs(p, seed=8)
    st = Stages(p, host)
    st.forward_unfused(); st.backward_unfused()
    nb = 2 * p.k - 1
    out = torch.empty((p.heads, nb, nb), dtype=torch.float32, device="cuda")
    na.na2d_qk_bwd_rpb_noalloc(st.ds, p.k, st.q, out)   # first use on the device: looks up the array's address
    torch.cuda.synchronize()
    assert torch.equal(out, st.d_rpb)
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        na.na2d_qk_bwd_rpb_noalloc(st.ds, p.k, st.q, out)
    for _ in range(3):
        out.fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, st.d_rpb)


def _replays_match(run, outs_of):
    """run() eagerly, then captured: four replays with eager work between them; every replay has the eager bits."""
    eager = [t.clone() for t in outs_of(run())]
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        outs = outs_of(run())
    for replay in range(4):
        for t in outs:
            t.fill_(float("nan"))
        other = [t.clone() for t in outs_of(run())]
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for i, (a, b, c) in enumerate(zip(outs, eager, other)):
            assert torch.equal(a, b) and torch.equal(c, b), f"replay {replay}: output {i}"


# wide windows in pairs of waves and alone, 64 channels, fp32
@pytest.mark.parametrize("B,H,W,D,k,dtype", [(2, 27, 41, 32, 21, "bf16"), (90, 17, 18, 32, 15, "f16"), (3, 19, 22, 64, 7, "f16"), (60, 14, 33, 32, 7, "f32")])
def test_direct_backward_under_capture(B, H, W, D, k, dtype):
    p = synth.Problem(B, 1, H, W, D, k, dtype)
    st = Stages(p, synth.make_inputs(p, seed=k))
    st.forward_fused()
    need = na.na2d_direct_bwd_workspace_bytes(na.problem(B, 1, H, W, D, k, st.tdtype))
    assert need > 0
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    grads = [torch.empty_like(st.q) for _ in range(3)] + [torch.empty((1, 2 * k - 1, 2 * k - 1), device="cuda")]

    def run():
        na.na2d_direct_bwd(st.q, st.key, st.v, st.rpb, st.scale, st.lse, st.dout, k, *grads, ws)
        return grads
    _replays_match(run, list)


@pytest.mark.parametrize("op,space,k,dtype", [(F.na2d, (14, 14), 7, "bf16"), (F.na2d, (22, 25), 13, "f16"), (F.na2d, (30, 33), 21, "bf16"), (F.na2d, (9, 13), 3, "f32"),
                                              (F.na1d, (311,), 7, "f16"), (F.na1d, (311,), 31, "f32"), (F.na2d_unfused, (14, 17), 5, "f16")])
def test_operators_under_capture(op, space, k, dtype):
    """The differentiable operators, forward and backward, in one graph."""
    torch.manual_seed(k)
    make = lambda *s: torch.randn(s, device="cuda").to(synth.TORCH_DTYPES[dtype])
    q, key, v = (make(3, 2, *space, 32).requires_grad_() for _ in range(3))
    rpb, dout = make(2, *(2 * k - 1 for _ in space)).requires_grad_(), make(3, 2, *space, 32)
    native = type(op(q, key, v, rpb, kernel_size=k).grad_fn).__name__

    def run():
        out = op(q, key, v, rpb, kernel_size=k)
        assert type(out.grad_fn).__name__ == native
        return (out.detach(), *torch.autograd.grad(out, (q, key, v, rpb), dout))
    _replays_match(run, list)
