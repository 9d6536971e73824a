"""Products of more than one turn whose eight row stripes give way to other regions of the tile grid (as many turns, and beyond two turns
7 % more tiles): ragged tile rows and columns in one, two and four stripes, compared with the oracle on sampled rows, codes and
accumulators bit for bit, Y and dX within the fp32 tolerance."""
import sys

import pytest

from paper_2505_14742_amd import binding as q
from paper_2505_14742_amd import synth

# (t, c_in, c_out, rank), direction, form
_CASES = [((197, 320, 1056, 48), 0, "32x32 rows"), ((398, 192, 528, 0), 0, "32x32 rows"), ((706, 320, 352, 48), 0, "32x32 rows"),
          ((462, 208, 4144, 48), 0, "64x128"), ((1481, 320, 3888, 48), 0, "64x128"), ((4110, 192, 1552, 48), 0, "64x128"),
          ((2827, 208, 2720, 48), 0, "128x192"), ((4614, 208, 1552, 16), 0, "128x192"), ((460, 4208, 192, 48), 2, "64x128"),
          ((1498, 3904, 208, 48), 2, "64x128"), ((4177, 1552, 192, 48), 2, "64x128"), ((2836, 2704, 208, 16), 2, "128x192")]


@pytest.mark.parametrize("shape,how,form", _CASES, ids=["%dx%dx%d_r%d" % c[0] for c in _CASES])
def test_form(shape, how, form):
    t, c_in, c_out, r = shape
    assert q.debug_product_form(t, c_in, c_out, 0, r, how) == form


@pytest.mark.gpu
@pytest.mark.parametrize("shape,how,form", _CASES, ids=["%dx%dx%d_r%d" % c[0] for c in _CASES])
def test_regions(shape, how, form):
    from tests.gpu_harness import Layer, OracleLayer, check_step, sample_rows
    t, c_in, c_out, r = shape
    print("regions", shape, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("regions", t, c_in, c_out, [5], r), 157)
    L, R = Layer(W, O, A if r else None, B if r else None, 1.0, t), OracleLayer(W, O, A if r else None, B if r else None, 1.0)
    check_step(L, R, X, dY, 0.2, rows=sample_rows(t, every=5), tag="regions %d x %d -> %d" % (t, c_in, c_out))
