"""The one-launch forward preparation hands column maxima between its workgroups through words of the caller's workspace.
Nothing that the workspace holds before a call may be taken for such a word: not what an earlier call wrote while its launch
counter had the value it has now, nor other data that agrees with the counter in a few bits.  The one call is compared with
the three separate calls bit for bit; the smallest workspace that is accepted must give the same bits too."""
import sys

import pytest

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

_FIELDS = ["s_O", "colscale", "what_int", "delta_what", "Xq", "delta_x", "xq_O", "Y"]
# (t, c_in, c_out, number of outliers, rank): two row owners and workgroups that only requantize what; owners alone, a last
# column without a partner; 255 owners and one more, an odd count of columns (the smallest workspace has no room for its words)
_CASES = [(16, 1040, 9216, 4, 16), (700, 512, 512, 1, 0), (2040, 4112, 4112, 3, 16)]


def _pair(t, c_in, c_out, n, r):
    import torch
    from tests.gpu_harness import Layer, bf16_dev
    ec = synth.EdgeCase("fwd_workspace", t, c_in, c_out, [9, c_in // 2, c_in - 1, 0][:n], r)
    print("forward workspace", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 41)
    loud = bf16_dev(X)                                  # outlier columns 50 times the others
    quiet = (loud.view(torch.bfloat16) * 2.0 ** -7).view(loud.dtype)
    return [Layer(W, O, A if r else None, B if r else None, 0.5, t) for _ in range(2)], loud, quiet


def _same_step(layers, X, call, tag):
    import torch
    three, one = layers
    three.scale_update(X, 0.2)
    three.quant_act(X)
    three.linear_fwd(X)
    call(one, X)
    torch.cuda.synchronize()
    for f in _FIELDS:
        assert torch.equal(getattr(three, f), getattr(one, f)), "%s: %s differs" % (tag, f)


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_what_the_workspace_held_does_not_matter(t, c_in, c_out, n, r):
    import torch
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV
    layers, loud, quiet = _pair(t, c_in, c_out, n, r)
    one = layers[1]
    ws = torch.zeros((q.fwd_step_workspace_bytes(t, c_in, c_out, one.n, r) + 7) // 8, dtype=torch.int64, device=DEV)
    one.ws_step, one.ws_step_t = ws.view(torch.int8), t
    step = lambda X, tag: _same_step(layers, X, lambda L, x: L.fwd_step(x, 0.2), tag)
    counts = torch.ones_like(ws, dtype=torch.bool)
    for call in (1, 2, 3):
        step(loud, "call %d" % call)
        counts &= ws == call
    at, = torch.nonzero(counts).flatten().tolist()       # the launch counter: 0, 1, 2, 3
    words = ws[at + 32:at + 32 + (one.n + 1) // 2 * 256]
    assert not words.any(), "words of a finished call are left"
    for again in range(3):
        # the counter as it was before the loud batch, as other calls on the same memory may leave it
        step(loud, "loud %d" % again)
        ws[at] -= 1
        step(quiet, "quiet %d, counter put back" % again)
    for pattern in ("lower half", "counter", "noise"):
        nxt = int(ws[at]) + 1
        if pattern == "lower half":
            words.view(torch.int32).fill_(0x7F000000 | nxt & 0xFFFF)
        elif pattern == "counter":
            words.fill_(nxt)
        else:
            words.view(torch.int32).random_(-2 ** 31, 2 ** 31 - 1)
        step(quiet, "words hold " + pattern)


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_smallest_workspace(t, c_in, c_out, n, r):
    import torch
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV, smallest_workspace
    layers, loud, quiet = _pair(t, c_in, c_out, n, r)
    one = layers[1]
    full = torch.empty(q.fwd_step_workspace_bytes(t, c_in, c_out, one.n, r), dtype=torch.int8, device=DEV)

    def call(L, X, size):
        L.ws_step, L.ws_step_t = full[:size], t
        L.fwd_step(X, 0.2)

    start = [x.clone() for x in (one.s_O, one.colscale)]
    small = smallest_workspace(lambda size: call(one, loud, size), full.numel())
    one.s_O.copy_(start[0])
    one.colscale.copy_(start[1])
    assert small < full.numel()
    for X in (loud, quiet):
        _same_step(layers, X, lambda L, x: call(L, x, small), "smallest workspace")
