"""Products of few rows or small outputs, whose wavefronts share the contraction: every tile shape in both directions (16 x 16,
32 x 32, 32 x 64 and 64 x 96 forward; 16 x 64 and 32 x 64 input gradient), ragged rows and columns, contractions shorter than
one step, not a multiple of a step and with fewer steps than wavefronts, every rank, no, one, several and many outlier
slices; compared with the oracle in full (accumulators bit for bit)."""
import sys

import pytest

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank)
_CASES = [(1, 208, 272, 5, 16), (33, 16, 16, 1, 48), (15, 80, 9232, 3, 64), (31, 272, 4112, 65, 32), (100, 3088, 1040, 130, 16),
          (48, 4112, 48, 300, 64), (65, 1040, 2064, 0, 0), (257, 1040, 2064, 13, 32), (193, 2064, 3088, 70, 16)]


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_rows_gemm(t, c_in, c_out, n, r):
    from tests.gpu_harness import Layer, OracleLayer, check_prepare, check_step
    O = [k * (c_in - 1) // max(n - 1, 1) for k in range(n)]
    ec = synth.EdgeCase("rows_gemm", t, c_in, c_out, O, r)
    print("rows gemm", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 93)
    L, R = Layer(W, O, A if r else None, B if r else None, 1.0, t), OracleLayer(W, O, A if r else None, B if r else None, 1.0)
    check_prepare(L, R)
    check_step(L, R, X, dY, 0.2, tag="rows gemm %d x %d x %d" % (t, c_in, c_out))
