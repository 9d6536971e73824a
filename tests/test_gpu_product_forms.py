"""Every kernel form that a product can take, in both directions: ragged rows, columns and contractions, no, one and two adapter staging
rounds, no, one, two and many outlier slices, each case with the form it is meant for asserted.  The reference is the same expression
in 64 bits from the same codes, scales and adapter; where bf16 results exist they are the fp32 results rounded."""
import sys

import pytest

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank), form of the forward product
_FORWARD = [
    ((1, 192, 208, 5, 16), "16x16 rows"), ((1, 192, 4720, 5, 32), "32x32 rows"), ((33, 960, 4720, 0, 16), "32x64 rows"),
    ((199, 192, 2544, 0, 32), "64x64"), ((1, 192, 8688, 70, 64), "64x64"), ((523, 192, 1584, 70, 0), "64x128"), ((132, 192, 5232, 70, 48), "64x128"),
    ((202, 192, 8816, 0, 0), "128x128"), ((4174, 848, 464, 70, 48), "128x128"), ((4194, 192, 1776, 70, 0), "128x192"),
    ((12450, 192, 544, 5, 32), "128x192"), ((9768, 192, 800, 0, 48), "128x192"), ((6312, 192, 528, 5, 32), "128x192 deep"),
    ((8227, 192, 400, 70, 64), "128x192 deep"), ((1077, 208, 4720, 0, 0), "256x128"), ((10747, 256, 416, 70, 32), "256x128"),
    ((1305, 208, 4384, 5, 64), "256x128"), ((4227, 192, 1200, 5, 0), "256x128 narrow"), ((2170, 192, 2576, 0, 64), "256x128 narrow"),
    ((5694, 192, 1968, 70, 32), "256x256"), ((12906, 208, 928, 70, 64), "256x256"), ((2328, 192, 4832, 0, 0), "256x256 narrow"),
    ((13091, 192, 944, 0, 48), "256x256 narrow"), ((2076, 208, 6608, 0, 16), "256x288"), ((13594, 192, 816, 5, 48), "256x288"),
    ((9051, 192, 1632, 0, 0), "256x288 narrow"), ((7293, 192, 1568, 0, 48), "256x288 narrow"), ((7426, 4160, 5968, 0, 0), "256x256 many"),
    ((6185, 4416, 6608, 5, 16), "256x256 many"),
    # many outliers: both contractions in one launch
    ((1, 192, 240, 175, 48), "64x64 wide"), ((94, 192, 8784, 156, 48), "64x128 wide"), ((585, 192, 3232, 192, 16), "128x128 wide"),
    ((8611, 448, 272, 275, 64), "128x128 wide"), ((11014, 240, 272, 240, 16), "128x192 deep wide"), ((3248, 192, 1168, 170, 48), "128x192 deep wide"),
    # ... or the main product accumulating onto the outliers' (the tiles of 64 and 128 rows do from 16384 columns on only)
    ((1, 928, 208, 293, 16), "16x16 rows onto 16x16 rows"), ((173, 2592, 608, 257, 16), "32x32 rows onto 32x32 rows"),
    ((17, 5744, 8224, 250, 48), "32x64 rows onto 32x32 rows"), ((1357, 8512, 6304, 141, 32), "128x192 onto 128x192"),
    ((12930, 8656, 528, 259, 64), "128x192 onto 128x192"), ((11668, 10048, 416, 568, 64), "256x128 narrow onto 256x128 narrow"),
    ((10250, 11264, 432, 140, 64), "256x128 onto 256x128 narrow"), ((10352, 1952, 1232, 204, 32), "256x256 onto 256x256"),
    ((1913, 1808, 6288, 290, 0), "256x256 onto 256x256 narrow"), ((8468, 3648, 1568, 221, 0), "256x288 onto 256x288"),
    ((3281, 2752, 4320, 221, 48), "256x288 onto 256x288"), ((2050, 2528, 6624, 265, 48), "256x288 onto 256x288 narrow"),
    ((35, 37472, 9344, 1589, 16), "64x64 onto 64x64"), ((198, 28336, 4400, 2414, 32), "64x128 onto 64x128"),
    ((134, 32944, 10976, 170, 64), "128x128 onto 128x128"), ((4132, 33424, 784, 1117, 64), "128x192 deep onto 64x128")]

# (t, c_in, c_out, rank), form of the input gradient
_GRADIENT = [
    ((1, 208, 224, 16), "16x64 rows"), ((17, 8800, 320, 16), "32x64 rows"), ((557, 208, 208, 32), "64x64"), ((67, 8992, 240, 16), "64x128"),
    ((65, 8240, 272, 64), "64x128"), ((212, 8240, 208, 32), "128x128"), ((6664, 272, 864, 48), "128x128"), ((6545, 1040, 208, 16), "128x192"),
    ((13454, 528, 224, 48), "128x192"), ((11723, 272, 224, 16), "128x192 deep"), ((11061, 272, 256, 48), "128x192 deep"),
    ((10545, 400, 208, 16), "256x128"), ((12901, 432, 192, 64), "256x128"), ((5484, 2016, 192, 32), "256x256"), ((7178, 1568, 224, 48), "256x256"),
    ((12779, 800, 240, 32), "256x288"), ((1665, 8544, 192, 48), "256x288"), ((7254, 5488, 4256, 16), "256x256 many"),
    ((11516, 3536, 4672, 0), "256x256 many"), ((1999, 3056, 12288, 16), "256x192 split")]


def _layer(t, c_in, c_out, n, r):
    """Codes, scales and adapter of one layer, drawn on the device."""
    import torch
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV
    gen = torch.Generator(device=DEV).manual_seed(t + 3 * c_in + 5 * c_out + 7 * n + r)
    W = torch.randn(c_in, c_out, generator=gen, device=DEV).mul_(0.02)
    L = {"Wq": torch.empty(q.packed_weight_bytes(c_in, c_out), dtype=torch.int8, device=DEV), "dw": torch.empty(c_out, device=DEV),
         "plain": torch.empty(c_in, c_out, dtype=torch.int8, device=DEV)}
    q.prepare_weight(W, None, L["Wq"], L["dw"], None, None, L["plain"],
                     torch.empty(q.prepare_workspace_bytes(c_in, c_out), dtype=torch.int8, device=DEV))
    L["A"] = (torch.randn(c_in, r, generator=gen, device=DEV) / c_in ** 0.5).to(torch.bfloat16) if r else None
    L["B"] = (torch.randn(r, c_out, generator=gen, device=DEV) * 0.02).to(torch.bfloat16) if r else None
    L["ws"] = torch.empty(q.workspace_bytes(t, c_in, c_out, n, r), dtype=torch.int8, device=DEV)
    return q, gen, L


def _compare(got, want):
    """The tolerance of 32-bit sums in another order and an adapter term kept in 16 significant bits: 4e-6 of the norm, 4e-5 of a value
    or, where that is larger, of the root mean square (see the same figures in perf/cases.py)."""
    diff = (got.double() - want).abs_()
    assert float(diff.norm() / want.norm()) <= 4e-6
    assert float((diff / want.abs().clamp(min=float(want.norm()) / want.numel() ** 0.5)).max()) <= 4e-5


@pytest.mark.parametrize("case,form", _FORWARD, ids=["%s_%dx%dx%d_n%d_r%d" % ((f.replace(" ", "_"),) + c) for c, f in _FORWARD])
def test_forward_form(case, form):
    import torch
    from tests.gpu_harness import DEV
    t, c_in, c_out, n, r = case
    print("forward form", form, case, flush=True)
    sys.stdout.flush()
    q, gen, L = _layer(*case)
    assert q.debug_product_form(*case, 0) == form
    X = torch.randn(t, c_in, generator=gen, device=DEV).to(torch.bfloat16)
    Xq, dx = torch.empty(t, c_in, dtype=torch.int8, device=DEV), torch.empty(t, device=DEV)
    q.quant_act(X, None, None, Xq, dx, None)
    n_pad = q.padded_outliers(n)
    xo, what, dwh = (None,) * 3
    if n:
        xo, what = (torch.randint(-127, 128, (rows, n_pad), generator=gen, device=DEV, dtype=torch.int8) for rows in (t, c_out))
        xo[:, n:] = 0
        what[:, n:] = 0
        dwh = torch.rand(c_out, generator=gen, device=DEV) * 1e-3

    def run(out, bf16):
        q.linear_fwd(Xq, dx, xo, L["Wq"], L["dw"], c_in, c_out, what, dwh, n, X if r else None, L["A"], L["B"], r, 0.5, out, L["ws"], bf16_out=bf16)
        return out

    Y = run(torch.full((t, c_out), float("nan"), device=DEV), False)
    want = (Xq.double() @ L["plain"].double()) * L["dw"].double()
    if n:
        want += (xo.double() @ what.double().T) * dwh.double()
    want *= dx.double()[:, None]
    if r:
        want += 0.5 * ((X.double() @ L["A"].double()) @ L["B"].double())
    _compare(Y, want)
    if c_in % 64 == 0 and n <= 128:
        assert torch.equal(run(torch.zeros(t, c_out, dtype=torch.bfloat16, device=DEV), True), Y.to(torch.bfloat16))


@pytest.mark.parametrize("case,form", _GRADIENT, ids=["%s_%dx%dx%d_r%d" % ((f.replace(" ", "_"),) + c) for c, f in _GRADIENT])
def test_gradient_form(case, form):
    import torch
    from tests.gpu_harness import DEV
    t, c_in, c_out, r = case
    print("gradient form", form, case, flush=True)
    sys.stdout.flush()
    q, gen, L = _layer(t, c_in, c_out, 0, r)
    assert q.debug_product_form(t, c_in, c_out, 0, r, 2) == form
    dY = (torch.randn(t, c_out, generator=gen, device=DEV) * 2.0 ** -6).to(torch.bfloat16)

    def run(out, bf16):
        q.linear_bwd_dx(dY, L["Wq"], L["dw"], c_in, c_out, L["A"], L["B"], r, 0.5, out, L["ws"], bf16_out=bf16)
        return out

    dX = run(torch.full((t, c_in), float("nan"), device=DEV), False)
    Gq, dg, acc = torch.empty(t, c_out, dtype=torch.int8, device=DEV), torch.empty(t, device=DEV), torch.empty(t, c_in, dtype=torch.int32, device=DEV)
    q.linear_bwd_dx_acc(dY, L["Wq"], L["dw"], c_in, c_out, Gq, dg, acc)
    sums = Gq.double() @ L["plain"].double().T
    assert torch.equal(acc.double(), sums)
    want = sums * dg.double()[:, None]
    if r:
        want += 0.5 * ((dY.double() @ L["B"].double().T) @ L["A"].double().T)
    _compare(dX, want)
    if c_out % 64 == 0:
        assert torch.equal(run(torch.zeros(t, c_in, dtype=torch.bfloat16, device=DEV), True), dX.to(torch.bfloat16))
