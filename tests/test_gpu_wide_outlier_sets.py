"""Requantization of what for more than 64 outlier channels: the number of outliers on both sides of each instantiation's
range (128, 256, 512, 1024 and 2048 held in registers, more fetched twice) and of a workgroup's thread count, dense sets and
sparse ones, few and odd numbers of output-channel groups, more groups than compute units, from one row to more rows than slabs; compared with the oracle (s, codes, scales and accumulators bit for bit) over two steps."""
import sys

import pytest

from paper_2505_14742_amd import synth

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers)
_CASES = [(1, 1040, 16, 65), (40, 8192, 48, 66), (300, 1040, 272, 256), (33, 1040, 80, 257), (17, 2064, 48, 512), (2100, 528, 16, 513),
          (64, 4112, 208, 819), (5, 1040, 48, 1023), (18, 1040, 32, 1025), (16, 2064, 80, 2048), (9, 2080, 48, 2049), (3, 4208, 16, 4160),
          (50, 1040, 4112, 128), (50, 1040, 4112, 129), (33, 1040, 4096, 256), (300, 272, 4128, 256)]


@pytest.mark.parametrize("t,c_in,c_out,n", _CASES, ids=["%dx%dx%d_n%d" % c for c in _CASES])
def test_wide_outlier_sets(t, c_in, c_out, n):
    from tests.gpu_harness import Layer, OracleLayer, check_prepare, check_step
    O = [k * (c_in - 1) // (n - 1) for k in range(n)]
    ec = synth.EdgeCase("wide_outlier_sets", t, c_in, c_out, O, 16)
    print("wide outlier sets", t, c_in, c_out, n, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(ec, 97)
    L, R = Layer(W, O, A, B, 1.0, t), OracleLayer(W, O, A, B, 1.0)
    check_prepare(L, R)
    for step in range(2):
        check_step(L, R, X, dY, 0.2, tag="%d outliers, step %d" % (n, step))
