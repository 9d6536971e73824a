"""LoRA weight gradients at the edges of the tiles of the gradient product: fewer tokens than a tile, a last tile of one token, the
largest count that is written without partial results and the smallest that is not, ragged last column chunks (128 columns a
workgroup at rank 16, 256 above), every rank, against the oracle."""
import pytest

from paper_2505_14742_amd import synth
from tests.test_gpu_lora_grads import _run

pytestmark = pytest.mark.gpu

_CASES = [(1, 16, 272, 16), (65, 144, 128, 16), (256, 400, 272, 16), (257, 128, 144, 16), (63, 256, 528, 32), (256, 16, 272, 48),
          (257, 528, 240, 48), (129, 272, 16, 64), (320, 240, 512, 64)]


@pytest.mark.parametrize("t,c_in,c_out,r", _CASES, ids=["%dx%dx%d_r%d" % c for c in _CASES])
def test_gradient_tiles(t, c_in, c_out, r):
    ec = synth.EdgeCase("grad_tiles", t, c_in, c_out, [], r)
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 94)
    _run(X, dY, A, B, 0.5, "gradient tiles")
