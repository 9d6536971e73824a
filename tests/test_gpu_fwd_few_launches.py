"""Which launches a forward step of few rows or columns makes, on both sides of the single launch's limits: 64 workgroups and 1024 columns
with outliers, 1024 gathered values, 256 workgroups and 2048 columns without (1024 without an adapter), ranks 0 and 16."""
import pytest

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

_ONE, _TWO = ["fwd_few"], ["fwd_prep", "gemm_i8"]
# (t, c_in, c_out, number of outliers, rank), launches
_CASES = [((16, 1024, 4096, 64, 16), _ONE), ((16, 1024, 4112, 2, 0), _TWO), ((16, 1040, 512, 1, 16), _TWO), ((64, 1024, 1024, 16, 0), _ONE),
          ((65, 1024, 192, 16, 0), _TWO), ((1, 2048, 4096, 0, 16), _ONE), ((15, 2064, 512, 0, 16), None), ((16, 1024, 16384, 0, 0), _ONE),
          ((16, 1024, 16400, 0, 0), None), ((15, 1040, 512, 0, 0), None), ((7, 320, 512, 0, 32), None)]


@pytest.mark.parametrize("shape,want", _CASES, ids=["%dx%dx%d_n%d_r%d" % c[0] for c in _CASES])
def test_launches(shape, want):
    import torch
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import Layer, bf16_dev
    t, c_in, c_out, n, r = shape
    O = sorted({k * (c_in - 1) // max(n - 1, 1) for k in range(n)})
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("few_launches", t, c_in, c_out, O, r), 163)
    L, Xd = Layer(W, O, A if r else None, B if r else None, 0.5, t), bf16_dev(X)
    L.fwd_step(Xd, 0.2)
    torch.cuda.synchronize()
    q.profile_enable(True)
    try:
        L.fwd_step(Xd, 0.2)
        torch.cuda.synchronize()
        kinds = [k for k, _ in q.profile_launches()]
    finally:
        q.profile_enable(False)
    if want is None:
        assert "fwd_few" not in kinds and len(kinds) >= 2, kinds
    else:
        assert kinds == want, kinds
