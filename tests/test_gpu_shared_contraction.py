"""Small outputs whose contraction two or four workgroups per tile share: ragged rows and columns, the fewest stages per part,
no, one and several outlier slices, every rank form, both directions; also with the bounded wait forced to give up, with a
workspace that has no room for the exchange, and several calls in a row on one workspace (the flags end at zero).  Integer
sums: exchanged and recomputed parts give the same bits."""
import sys

import pytest
import torch

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank): four parts forward; two; two in the gradient; ragged edges with both; four
# parts in the gradient, whole and ragged
_CASES = [(257, 8192, 3056, 1, 16), (512, 3072, 3072, 31, 16), (500, 3088, 4096, 70, 48), (129, 8192, 6160, 0, 0),
          (1000, 4096, 3008, 65, 64), (384, 4096, 8192, 13, 32),
          (256, 4096, 4096, 5, 16), (257, 3056, 8192, 31, 32)]


def _forward(q, L, X, dY, ws):
    Y = torch.full((L.t, L.c_out), -3.0, device=X.device)
    q.linear_fwd(L.Xq, L.delta_x, L.xq_O, L.Wq_packed, L.delta_w, L.c_in, L.c_out, L.what_int if L.n else None,
                 L.delta_what if L.n else None, L.n, X if L.r else None, L.A, L.B, L.r, L.lora_scale, Y, ws)
    return Y


def _gradient(q, L, X, dY, ws):
    dX = torch.full((L.t, L.c_in), -3.0, device=X.device)
    q.linear_bwd_dx(dY, L.Wq_packed, L.delta_w, L.c_in, L.c_out, L.A, L.B, L.r, L.lora_scale, dX, ws)
    return dX


def _outputs(q, L, X, dY, ws):
    return _forward(q, L, X, dY, ws), _gradient(q, L, X, dY, ws)


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_shared_contraction(t, c_in, c_out, n, r):
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import Layer, bf16_dev, smallest_workspace
    O = [k * (c_in - 1) // max(n - 1, 1) for k in range(n)]
    print("shared contraction", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("shared_contraction", t, c_in, c_out, O, r), 101)
    L = Layer(W, O, A if r else None, B if r else None, 1.0, t)
    Xd, dYd = bf16_dev(X), bf16_dev(dY)
    L.fwd_step(Xd, 0.2)
    ws = torch.empty(q.workspace_bytes(t, c_in, c_out, n, r), dtype=torch.int8, device=Xd.device)
    # the smallest workspace that each call accepts holds no exchange area: one workgroup per tile
    alone = []
    for call in (_forward, _gradient):
        small = smallest_workspace(lambda size: call(q, L, Xd, dYd, ws[:size]), ws.numel())
        assert small < ws.numel()
        alone.append(call(q, L, Xd, dYd, ws[:small]))
    prev = q.debug_grid_wait_ticks(0)
    try:
        want = _outputs(q, L, Xd, dYd, ws)                # every workgroup may give up and compute all parts itself
    finally:
        q.debug_grid_wait_ticks(prev)
    for attempt in range(4):
        got = _outputs(q, L, Xd, dYd, ws)
        assert all(torch.equal(a, b) for a, b in zip(got, want)), "attempt %d" % attempt
    assert all(torch.equal(a, b) for a, b in zip(alone, want)), "alone"


def _steps(t, c_in, c_out, r):
    """A layer, its inputs and a backward step on a workspace and outputs of its own; forward step from the layer."""
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV, Layer, bf16_dev
    print("shared contraction, steps", t, c_in, c_out, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("shared_steps", t, c_in, c_out, [2, c_in - 3], r), 103)
    L = Layer(W, O, A, B, 1.0, t)
    Xd, dYd = bf16_dev(X), bf16_dev(dY)
    ws = torch.empty(q.bwd_step_workspace_bytes(t, c_in, c_out, r), dtype=torch.int8, device=DEV)
    out = [torch.empty(s, device=DEV) for s in ((t, c_in), (c_in, r), (r, c_out))]

    def backward(side, ws=ws):
        q.linear_bwd_step(dYd, Xd, L.Wq_packed, L.delta_w, c_in, c_out, L.A, L.B, r, 1.0, *out, ws, side=side)
        return [x.clone() for x in out]

    return q, L, Xd, dYd, ws, backward


# four parts (and weight gradients whose workgroups leave no room beside the sharing ones: rank 64), two parts, ragged; two parts
# that are not worth it beside such weight gradients
_STEPS = [(256, 4096, 4096, 64), (512, 3072, 3072, 16), (257, 3056, 8192, 32), (1900, 1536, 4096, 32)]


@pytest.mark.parametrize("t,c_in,c_out,r", _STEPS, ids=["%dx%dx%d_r%d" % c for c in _STEPS])
def test_shared_contraction_in_the_backward_step(t, c_in, c_out, r):
    """Behind the weight gradients' area of the workspace, alone and beside a second stream that fills the chip, with the wait
    as it is and forced to give up, and without room for the exchange: the bits of quaff_linear_bwd_dx."""
    from tests.gpu_harness import smallest_workspace
    q, L, Xd, dYd, ws, backward = _steps(t, c_in, c_out, r)
    L.linear_bwd_dx(dYd)
    first = backward(None)
    small = smallest_workspace(lambda size: backward(None, ws[:size]), ws.numel())
    assert small < ws.numel()
    side = q.SideStream()
    prev = q.debug_grid_wait_ticks(-1)
    for ticks in (prev, 0):
        q.debug_grid_wait_ticks(ticks)
        try:
            for again in range(3):
                for how, got in (("one stream", backward(None)), ("second stream", backward(side)),
                                 ("no room", backward(side, ws[:small]))):
                    tag = "%s, wait %d, %d" % (how, ticks, again)
                    assert torch.equal(got[0], L.dX), tag
                    assert torch.equal(got[1], first[1]) and torch.equal(got[2], first[2]), tag
        finally:
            q.debug_grid_wait_ticks(prev)


def test_shared_contraction_in_a_captured_step():
    """A forward and a backward step whose products share their contraction, captured once and replayed between eager steps on
    the same workspaces: every replay gives the bits of the eager step from the same state."""
    q, L, Xd, dYd, ws, backward = _steps(512, 3072, 3072, 16)
    side = q.SideStream()

    def step():
        L.fwd_step(Xd, 0.2)
        return [L.Y, L.s_O] + backward(side)

    start = [L.s_O.clone(), L.colscale.clone()]

    def rewind():
        L.s_O.copy_(start[0])
        L.colscale.copy_(start[1])

    step()
    rewind()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = step()
    for replay in range(4):
        rewind()
        want = [x.clone() for x in step()]
        rewind()
        L.Y.fill_(float("nan"))
        graph.replay()
        torch.cuda.synchronize()
        for name, a, b in zip(("Y", "s_O", "dX", "dA", "dB"), captured, want):
            assert torch.equal(a, b), "replay %d: %s" % (replay, name)
