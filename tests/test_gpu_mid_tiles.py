"""Outputs that take the tiles of 64 x 64, 64 x 128 and 128 x 128 (each in both directions below), with ragged rows, columns and
contractions, more tiles than compute units, every rank, no, one, several and many outlier slices; compared with the oracle in
full (accumulators bit for bit).  Then the 128 x 192 tile with eight and with four wavefronts (the backward step beside a second
stream): the same bits."""
import sys

import pytest
import torch

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank) and the tiles of the forward product and the input gradient
_CASES = [(500, 3056, 3088, 1, 16),     # 64 x 128, 64 x 128
          (241, 1360, 4112, 70, 64),    # 64 x 128, 64 x 64
          (1003, 1040, 2064, 13, 32),   # 128 x 128, 64 x 128
          (1290, 2032, 1936, 5, 48),    # 128 x 128, 128 x 128
          (192, 1216, 3600, 0, 0),      # 64 x 64, none of them
          (900, 2704, 3216, 130, 16),   # 128 x 128 (both contractions in one launch), 128 x 128
          (449, 1296, 1680, 2, 32),     # 64 x 64, 64 x 64
          (64, 208, 16016, 3, 16)]      # one tile row, 126 columns of tiles


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_mid_tiles(t, c_in, c_out, n, r):
    from tests.gpu_harness import Layer, OracleLayer, check_prepare, check_step
    O = [k * (c_in - 1) // max(n - 1, 1) for k in range(n)]
    ec = synth.EdgeCase("mid_tiles", t, c_in, c_out, O, r)
    print("mid tiles", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 131)
    L, R = Layer(W, O, A if r else None, B if r else None, 1.0, t), OracleLayer(W, O, A if r else None, B if r else None, 1.0)
    check_prepare(L, R)
    check_step(L, R, X, dY, 0.2, tag="mid tiles %d x %d x %d" % (t, c_in, c_out))


# more than two slices of outliers: summed in the product's launch on the tiles of 128 x 192, 128 x 128, 64 x 128 and 64 x 64, an odd
# and an even number of slices; in a launch of its own that the product accumulates onto (few rows)
_WIDE = [(1990, 336, 3056, 190, 48), (900, 528, 3216, 150, 16), (300, 528, 4128, 210, 48), (240, 1040, 1040, 140, 32), (1500, 272, 2064, 271, 0),
         (48, 4112, 48, 300, 64)]


@pytest.mark.parametrize("t,c_in,c_out,n,r", _WIDE, ids=["%dx%dx%d_n%d_r%d" % c for c in _WIDE])
def test_wide_outlier_products(t, c_in, c_out, n, r):
    test_mid_tiles(t, c_in, c_out, n, r)


@pytest.mark.parametrize("t,c_in,c_out,r", [(2048, 3072, 1024, 16), (1999, 3056, 784, 48)])
def test_deep_tile_beside_a_second_stream(t, c_in, c_out, r):
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV, Layer, bf16_dev
    print("deep tile, second stream", t, c_in, c_out, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("deep_tile", t, c_in, c_out, [2, c_in - 3], r), 133)
    L = Layer(W, O, A, B, 1.0, t)
    Xd, dYd = bf16_dev(X), bf16_dev(dY)
    L.linear_bwd_dx(dYd)
    ws = torch.empty(q.bwd_step_workspace_bytes(t, c_in, c_out, r), dtype=torch.int8, device=DEV)
    out = [torch.empty(s, device=DEV) for s in ((t, c_in), (c_in, r), (r, c_out))]
    side = q.SideStream()
    for how in (None, side, side):
        for x in out:
            x.fill_(-3.0)
        q.linear_bwd_step(dYd, Xd, L.Wq_packed, L.delta_w, c_in, c_out, L.A, L.B, r, 1.0, *out, ws, side=how)
        assert torch.equal(out[0], L.dX)


@pytest.mark.parametrize("r", [0, 16])
def test_many_large_tiles(r):
    """More than 512 tiles of 256 x 256, sixteen wavefronts each (ragged rows, columns and contraction): without an adapter the bits of
    the same rows in a product of few tiles; with one, whose products may be added in another order there, 1e-6 of the result."""
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV
    t, c_in, c_out = 8447, 4112, 5104
    print("many large tiles", r, flush=True)
    sys.stdout.flush()
    gen = torch.Generator(device=DEV).manual_seed(7)
    W = torch.randn(c_in, c_out, generator=gen, device=DEV) * 0.02
    Wq, dw = torch.empty(q.packed_weight_bytes(c_in, c_out), dtype=torch.int8, device=DEV), torch.empty(c_out, device=DEV)
    q.prepare_weight(W, None, Wq, dw, None, None, None, torch.empty(q.prepare_workspace_bytes(c_in, c_out), dtype=torch.int8, device=DEV))
    X = torch.randn(t, c_in, generator=gen, device=DEV).to(torch.bfloat16)
    A = (torch.randn(c_in, r, generator=gen, device=DEV) / 64).to(torch.bfloat16) if r else None
    B = (torch.randn(r, c_out, generator=gen, device=DEV) * 0.02).to(torch.bfloat16) if r else None
    ws = torch.empty(q.workspace_bytes(t, c_in, c_out, 0, r), dtype=torch.int8, device=DEV)

    def forward(x):
        n = x.shape[0]
        Xq, d = torch.empty(n, c_in, dtype=torch.int8, device=DEV), torch.empty(n, device=DEV)
        q.quant_act(x, None, None, Xq, d, None)
        Y = torch.full((n, c_out), -3.0, device=DEV)
        q.linear_fwd(Xq, d, None, Wq, dw, c_in, c_out, None, None, 0, x if r else None, A, B, r, 1.0, Y, ws)
        return Y

    whole, parts = forward(X), torch.cat([forward(X[i:i + 300]) for i in range(0, t, 300)])
    if r == 0:
        assert torch.equal(whole, parts)
    else:
        assert float((whole.double() - parts.double()).norm() / parts.double().norm()) <= 1e-6
