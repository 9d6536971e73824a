"""The backward preparation with one and with two workgroups to a compute unit: both sides of its limits (1024 rows at rank 16, 4096 at
rank 32, 8192 columns) and every number of vectors a row, ragged rows: the codes and scales of the separate quantizer, bit for bit, and the
gradients of the oracle."""
import pytest

from paper_2505_14742_amd import synth
from tests.test_gpu_bwd_step import _run

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, rank)
_CASES = [(1023, 208, 5136, 16), (1024, 208, 5136, 16), (1037, 272, 8192, 16), (1030, 208, 8208, 16), (4096, 208, 208, 32),
          (4097, 208, 1024, 32), (4101, 208, 1040, 32), (4099, 224, 2064, 32), (4111, 208, 3088, 32), (4098, 208, 4112, 32),
          (4097, 208, 8192, 32), (4097, 208, 8208, 32)]


@pytest.mark.parametrize("t,c_in,c_out,r", _CASES, ids=["%dx%dx%d_r%d" % c for c in _CASES])
def test_backward_step(t, c_in, c_out, r):
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("bwd_prep", t, c_in, c_out, [1], r), 151)
    _run(W, O, A, B, 0.5, X, dY, "pairs t=%d %d -> %d r=%d" % (t, c_out, c_in, r))


@pytest.mark.parametrize("t,c_in,c_out,r", _CASES[2::5], ids=["%dx%dx%d_r%d" % c for c in _CASES[2::5]])
def test_codes(t, c_in, c_out, r):
    from tests.gpu_harness import Layer, OracleLayer, check_step, sample_rows
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("bwd_prep", t, c_in, c_out, [1], r), 153)
    check_step(Layer(W, O, A, B, 0.5, t), OracleLayer(W, O, A, B, 0.5), X, dY, 0.2, rows=sample_rows(t), tag="pairs")
