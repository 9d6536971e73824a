"""Backward quantizer whose workgroup shares eight long rows (ranks 48 and 64, more than 2048 rows): ragged row counts, the
shortest and longest rows it takes, rows that end inside a wavefront, a leading dimension of its own, zero rows.  With a zero
adapter the input gradient is that of the call without one, which takes the stand-alone quantizer (the products may round
their few fp32 operations in another order: 1e-6), and the low-rank part is checked in 64 bits."""
import sys

import pytest
import torch

pytestmark = pytest.mark.gpu

_CASES = [(2049, 4112, 48, 0), (2063, 8192, 64, 0), (2056, 8208, 64, 8), (2100, 16384, 48, 0), (2055, 11008, 64, 64), (2048, 8208, 64, 0)]


@pytest.mark.parametrize("t,c_out,r,pad", _CASES, ids=["%dx%d_r%d_pad%d" % c for c in _CASES])
def test_shared_rows(t, c_out, r, pad):
    from paper_2505_14742_amd import binding as q
    print("shared rows", t, c_out, r, pad, flush=True)
    sys.stdout.flush()
    dev, c_in = "cuda", 272
    gen = torch.Generator(device=dev).manual_seed(t + c_out)
    W = torch.randn(c_in, c_out, generator=gen, device=dev) * 0.02
    Wq = torch.empty(q.packed_weight_bytes(c_in, c_out), dtype=torch.int8, device=dev)
    dw = torch.empty(c_out, device=dev)
    q.prepare_weight(W, None, Wq, dw, None, None, None, torch.empty(q.prepare_workspace_bytes(c_in, c_out), dtype=torch.int8, device=dev))
    dY = torch.randn(t, c_out + pad, generator=gen, device=dev).mul_(2.0 ** -6).to(torch.bfloat16)[:, :c_out]
    dY[5] = 0
    A = (torch.randn(c_in, r, generator=gen, device=dev) / c_in ** 0.5).to(torch.bfloat16)
    B = (torch.randn(r, c_out, generator=gen, device=dev) * 0.02).to(torch.bfloat16)
    ws = torch.empty(q.workspace_bytes(t, c_in, c_out, 0, r), dtype=torch.int8, device=dev)

    def gradient(a, b, rank):
        dX = torch.full((t, c_in), float("nan"), device=dev)
        q.linear_bwd_dx(dY, Wq, dw, c_in, c_out, a, b, rank, 1.0, dX, ws)
        return dX.double()

    plain = gradient(None, None, 0)
    zero = gradient(A, torch.zeros_like(B), r)
    assert float((zero - plain).norm() / plain.norm()) <= 1e-6
    low = dY.double() @ B.double().T @ A.double().T
    full = gradient(A, B, r)
    # the intermediate keeps 16 significant bits (hi and lo bf16 parts): 2^-16 of it, and fp32 sums
    assert float((full - plain - low).norm() / low.norm()) <= 4e-5
