"""Small outputs whose contraction two or four workgroups per tile share: ragged rows and columns, the fewest stages per part,
no, one and several outlier slices, every rank form, both directions; also with the bounded wait forced to give up, with a
workspace that has no room for the exchange, and several calls in a row on one workspace (the flags end at zero).  Integer
sums: exchanged and recomputed parts give the same bits."""
import sys

import pytest
import torch

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank) and the parts of the forward product and the input gradient: ragged rows and columns, no,
# one and two outlier slices, every rank form
_CASES = [((195, 10752, 2208, 1, 16), 4, 1), ((203, 8704, 2096, 0, 0), 4, 1), ((2090, 11264, 912, 70, 16), 2, 1),
          ((646, 14336, 2736, 65, 48), 2, 1), ((323, 13312, 1296, 13, 64), 4, 1), ((212, 10752, 2112, 31, 32), 4, 1),
          ((198, 2112, 13824, 5, 16), 1, 4), ((917, 2064, 6144, 31, 32), 1, 2), ((527, 1680, 11264, 0, 0), 1, 2),
          ((685, 2768, 11264, 3, 48), 1, 2), ((208, 2064, 15872, 2, 64), 1, 4), ((65, 8704, 10752, 2, 16), 4, 4)]
# long and medium contractions that are faster unshared: the size of the workspace makes no difference
_CASES += [(case, 1, 1) for case in [(257, 8192, 3056, 1, 16), (512, 3072, 3072, 31, 16), (500, 3088, 4096, 70, 48), (129, 8192, 6160, 0, 0),
                                     (1000, 4096, 3008, 65, 64), (384, 4096, 8192, 13, 32), (256, 4096, 4096, 5, 16), (257, 3056, 8192, 31, 32)]]


def _parts(form):
    return int(form.rsplit(" ", 1)[1]) if "shared by" in form else 1


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


@pytest.mark.parametrize("case,forward,gradient", _CASES, ids=["%dx%dx%d_n%d_r%d" % c[0] for c in _CASES])
def test_shared_contraction(case, forward, gradient):
    t, c_in, c_out, n, r = case
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import Layer, bf16_dev, smallest_workspace
    assert [_parts(q.debug_product_form(*case, how)) for how in range(4)] == [forward, 1, gradient, 1]
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


# (t, c_in, c_out, rank), parts alone and beside a second stream: four and two parts that are worth it beside the weight gradients of
# every rank (at rank 32 and more these leave the sharing workgroups no room on a unit) and that are not, ragged
_STEPS = [((647, 2864, 6144, 16), 2, 2), ((202, 2064, 14336, 16), 4, 4), ((662, 2720, 10240, 32), 2, 2), ((917, 2064, 6144, 32), 2, 1),
          ((200, 2112, 13824, 32), 4, 1), ((792, 1040, 15360, 32), 4, 4), ((700, 2832, 16384, 64), 2, 2), ((650, 3040, 10752, 64), 2, 1),
          ((788, 1072, 15360, 64), 4, 4), ((208, 2064, 15872, 64), 4, 1)]
_STEPS += [(case, 1, 1) for case in [(256, 4096, 4096, 64), (512, 3072, 3072, 16), (257, 3056, 8192, 32), (1900, 1536, 4096, 32)]]


@pytest.mark.parametrize("case,alone,beside", _STEPS, ids=["%dx%dx%d_r%d" % c[0] for c in _STEPS])
def test_shared_contraction_in_the_backward_step(case, alone, beside):
    """Behind the weight gradients' area of the workspace, alone and beside a second stream that fills the chip, with the wait
    as it is and forced to give up, and without room for the exchange: the bits of quaff_linear_bwd_dx."""
    from tests.gpu_harness import smallest_workspace
    t, c_in, c_out, r = case
    q, L, Xd, dYd, ws, backward = _steps(t, c_in, c_out, r)
    assert [_parts(q.debug_product_form(t, c_in, c_out, 2, r, how)) for how in (2, 3, 4)] == [alone, 1, beside]
    L.linear_bwd_dx(dYd)
    first = backward(None)
    small = smallest_workspace(lambda size: backward(None, ws[:size]), ws.numel())
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
    t, c_in, c_out, r = 66, 8704, 10752, 16
    q, L, Xd, dYd, ws, backward = _steps(t, c_in, c_out, r)
    assert [_parts(q.debug_product_form(t, c_in, c_out, 2, r, how)) for how in (0, 4)] == [4, 4]
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
