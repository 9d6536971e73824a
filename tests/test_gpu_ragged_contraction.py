"""Products whose contraction is not a whole number of 128-byte stages, in both directions (forward over c_in, input
gradient over c_out): remainders of 16 to 112 bytes, contractions shorter than a stage and shorter than the ring, one
product per tile shape, compared with the oracle in full (accumulators bit for bit)."""
import sys

import pytest

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# stages of (forward, gradient): 1 and 1; 1 and 2; 2 and 3; 3 and 4; 9 and 17; 256-row tiles; 128 x 192 tiles, ring of three
_CASES = [(70, 16, 16), (130, 112, 144), (300, 144, 272), (520, 304, 400), (257, 1040, 2064), (2600, 208, 9232),
          (2048, 336, 3056)]


# forward contractions of whole 64-byte stages, an odd number of them: 1, 3, 5, 7, 11 and 17 stages and the ring of four or three;
# 128 x 192, 256 x 128, 256 x 256 and 256 x 288 tiles with edges and without; more than 128 outliers (a second launch adds up);
# no outliers, where the two largest tiles take these stages
_HALF = [(1530, 64, 3056, 2), (2048, 192, 3072, 2), (2001, 704, 2064, 2), (2050, 320, 9216, 2), (8192, 1088, 1024, 2),
         (4000, 192, 8000, 2), (2000, 320, 9104, 2), (1530, 448, 3056, 150), (4000, 192, 8000, 0),
         (2000, 320, 9104, 0), (2000, 960, 9104, 0)]


@pytest.mark.parametrize("t,c_in,c_out,n", _HALF, ids=["%dx%dx%d_n%d" % c for c in _HALF])
def test_half_a_stage_more(t, c_in, c_out, n):
    test_ragged_contraction(t, c_in, c_out, n)


@pytest.mark.parametrize("t,c_in,c_out", _CASES, ids=["%dx%dx%d" % c for c in _CASES])
def test_ragged_contraction(t, c_in, c_out, n=2):
    from tests.gpu_harness import Layer, OracleLayer, check_prepare, check_step
    O = [1, c_in - 1] if n == 2 else list(range(1, 2 * n, 2))
    ec = synth.EdgeCase("ragged_contraction", t, c_in, c_out, O, 16)
    print("ragged contraction", t, c_in, c_out, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 92)
    L, R = Layer(W, O, A, B, 1.0, t), OracleLayer(W, O, A, B, 1.0)
    check_prepare(L, R)
    check_step(L, R, X, dY, 0.2, tag="ragged contraction %d x %d x %d" % (t, c_in, c_out))
