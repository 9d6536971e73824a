"""Small outputs whose contraction two or four workgroups per tile share: ragged rows and columns, the fewest stages per part,
no, one and several outlier slices, every rank form, both directions; also with the bounded wait forced to give up, with a
workspace that has no room for the exchange, and several calls in a row on one workspace (the flags end at zero).  Integer
sums: exchanged and recomputed parts give the same bits."""
import sys

import pytest
import torch

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank): four parts forward; two; two in the gradient; ragged edges with both
_CASES = [(257, 8192, 3056, 1, 16), (512, 3072, 3072, 31, 16), (500, 3088, 4096, 70, 48), (129, 8192, 6160, 0, 0),
          (1000, 4096, 3008, 65, 64), (384, 4096, 8192, 13, 32)]


def _outputs(q, L, X, dY, ws):
    L.Y.fill_(-3.0)
    q.linear_fwd(L.Xq, L.delta_x, L.xq_O, L.Wq_packed, L.delta_w, L.c_in, L.c_out, L.what_int if L.n else None,
                 L.delta_what if L.n else None, L.n, X if L.r else None, L.A, L.B, L.r, L.lora_scale, L.Y, ws)
    dX = torch.full((L.t, L.c_in), -3.0, device=X.device)
    q.linear_bwd_dx(dY, L.Wq_packed, L.delta_w, L.c_in, L.c_out, L.A, L.B, L.r, L.lora_scale, dX, ws)
    return L.Y.clone(), dX


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_shared_contraction(t, c_in, c_out, n, r):
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import Layer, bf16_dev
    O = [k * (c_in - 1) // max(n - 1, 1) for k in range(n)]
    print("shared contraction", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("shared_contraction", t, c_in, c_out, O, r), 101)
    L = Layer(W, O, A if r else None, B if r else None, 1.0, t)
    Xd, dYd = bf16_dev(X), bf16_dev(dY)
    L.fwd_step(Xd, 0.2)
    # the smallest workspaces that were ever accepted hold no exchange area: the unsplit products
    full = q.workspace_bytes(t, c_in, c_out, n, r)
    ws = torch.empty(full, dtype=torch.int8, device=Xd.device)
    room = lambda size: ws[:size]
    lo, hi = 0, full
    while lo < hi:                       # the smallest size that both calls accept
        mid = (lo + hi) // 2
        try:
            _outputs(q, L, Xd, dYd, room(mid))
            hi = mid
        except Exception:
            lo = mid + 1
    alone = _outputs(q, L, Xd, dYd, room(lo))
    prev = q.debug_grid_wait_ticks(0)
    try:
        want = _outputs(q, L, Xd, dYd, ws)                # every workgroup may give up and compute all parts itself
    finally:
        q.debug_grid_wait_ticks(prev)
    for attempt in range(4):
        got = _outputs(q, L, Xd, dYd, ws)
        assert all(torch.equal(a, b) for a, b in zip(got, want)), "attempt %d" % attempt
    # (the unsplit product may be another kernel, whose epilogue rounds its few fp32 operations in another order)
    for a, b in zip(alone, want):
        assert float((a - b).double().norm() / b.double().norm()) <= 1e-6
