"""One-launch forward preparation with fewer row owners than compute units: the launch may be filled up with workgroups that
only requantize what.  Token counts on both sides of each way the channels are shared out (rounds of 64 channels: one per
extra workgroup, two, an equal share for everybody, the owners alone), ragged rows and channels, with and without an
adapter; the one call against the three separate calls bit for bit, also with the grid-wide wait forced to give up."""
import sys

import pytest

from paper_2505_14742_amd import synth
from tests.test_gpu_fwd_step import _compare

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, rank): one owner and an extra workgroup for each round; an equal share for everybody (256 rounds and 128
# workgroups, 144 and 128); a single round; owners alone: 193, 255 and 256 of them
_CASES = [(1, 256, 9232, 16), (16, 1040, 16384, 0), (9, 64, 16, 16), (1000, 256, 9216, 16), (1537, 128, 9232, 0),
          (2040, 128, 4112, 16), (2041, 128, 4112, 16)]


@pytest.mark.parametrize("wait", ["waits", "gives_up"])
@pytest.mark.parametrize("t,c_in,c_out,r", _CASES, ids=["%dx%dx%d_r%d" % c for c in _CASES])
def test_few_rows(t, c_in, c_out, r, wait):
    from paper_2505_14742_amd import binding as q
    ec = synth.EdgeCase("few_rows", t, c_in, c_out, [0, 5, 31, c_in - 1], r)
    print("few rows", t, c_in, c_out, r, wait, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 91)
    prev = q.debug_grid_wait_ticks(0) if wait == "gives_up" else None
    try:
        _compare(W, O, A if r else None, B if r else None, 0.5, [X, X[::-1].copy()], 0.2, "few rows t=%d" % t)
    finally:
        if prev is not None:
            q.debug_grid_wait_ticks(prev)


# how far the launch is filled up: to 128 workgroups with two rounds each and with an equal share for everybody, to 192, to
# 128 just beyond that; few rounds; short rows whose owners have a round each at most, owners alone; 128 and 129 owners.  Up to
# 256 with long rows: 255 owners and one extra, 128 extras with two rounds each, an equal share, no room.  Owners alone and
# filled up on either side of 768 columns, and with two rounds for 64 and for 63 owners
_FILLS = [(128, 128, 12800, 16), (500, 1040, 9216, 16), (64, 272, 10240, 0), (72, 272, 7696, 16), (40, 4112, 1040, 16),
          (260, 1040, 2064, 16), (384, 1024, 3072, 16), (1024, 128, 9232, 0), (1030, 128, 9232, 16),
          (2040, 4112, 4112, 16), (1024, 4112, 9232, 16), (1800, 4112, 9232, 0), (2041, 4112, 4112, 0),
          (64, 768, 512, 16), (64, 752, 512, 16), (512, 1024, 8192, 16), (504, 1024, 8192, 0)]


@pytest.mark.parametrize("wait", ["waits", "gives_up"])
@pytest.mark.parametrize("t,c_in,c_out,r", _FILLS, ids=["%dx%dx%d_r%d" % c for c in _FILLS])
def test_how_far_filled(t, c_in, c_out, r, wait):
    test_few_rows(t, c_in, c_out, r, wait)
