"""Forward steps of few rows or columns in a single launch against the three separate calls, bit for bit: both sides of its limits
(256 and 64 workgroups, 2048 and 1024 columns, 1024 gathered values), every number of slices per wavefront, tiles of 16, 32 and 64
channels, ragged rows, channels and contractions, no outliers and as many as fit; repeated on one workspace, whose words must be
zeros again and whose counter advances by one a call."""
import sys

import pytest

from paper_2505_14742_amd import synth
from tests.test_gpu_fwd_step import _compare

pytestmark = pytest.mark.gpu

# (t, c_in, c_out, number of outliers, rank)
_CASES = [(1, 16, 16, 1, 16), (7, 64, 48, 3, 0), (16, 80, 1024, 64, 16), (16, 208, 1040, 5, 0), (17, 320, 512, 9, 16), (16, 1024, 4096, 64, 16),
          (16, 1024, 4112, 2, 0), (64, 1024, 1024, 16, 0), (65, 1024, 192, 15, 16), (16, 1040, 512, 1, 16), (500, 256, 112, 2, 0),
          (1, 2048, 4096, 0, 16), (250, 2032, 1008, 0, 0), (33, 1056, 272, 0, 16), (16, 1536, 16400, 0, 0), (15, 2064, 512, 0, 0)]


@pytest.mark.parametrize("t,c_in,c_out,n,r", _CASES, ids=["%dx%dx%d_n%d_r%d" % c for c in _CASES])
def test_fwd_few(t, c_in, c_out, n, r):
    O = sorted({k * (c_in - 1) // max(n - 1, 1) for k in range(n)})
    print("few", t, c_in, c_out, n, r, flush=True)
    sys.stdout.flush()
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("fwd_few", t, c_in, c_out, O, r), 137)
    _compare(W, O, A if r else None, B if r else None, 0.5, [X, X[::-1].copy(), X], 0.2, "few t=%d" % t)


def test_words_and_counter():
    import torch
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV, Layer, bf16_dev
    t, c_in, c_out, r = 40, 512, 320, 16
    X, dY, W, O, A, B = synth.edge_case_inputs(synth.EdgeCase("fwd_few_words", t, c_in, c_out, [1, 77, 511], r), 139)
    L, Xd = Layer(W, O, A, B, 0.5, t), bf16_dev(X)
    ws = torch.zeros((q.fwd_step_workspace_bytes(t, c_in, c_out, L.n, r) + 7) // 8, dtype=torch.int64, device=DEV)
    L.ws_step, L.ws_step_t = ws.view(torch.int8), t
    for call in range(1, 6):
        L.fwd_step(Xd, 0.2)
        assert ws.count_nonzero() == 1 and int(ws.max()) == call
    # marks of a launch that the counter repeats, and noise: neither counts as a workgroup's
    state = [x.clone() for x in (L.s_O, L.colscale)]
    at = int(ws.argmax())
    for fill in (0, 1, 2):
        ws[at + 32:at + 32 + 256].fill_(-1 if fill == 1 else 0)
        if fill == 2:
            ws[at + 32:at + 32 + 256].view(torch.int32).random_(-2 ** 31, 2 ** 31 - 1)
        L.s_O.copy_(state[0])
        L.colscale.copy_(state[1])
        L.fwd_step(Xd, 0.2)
        if fill == 0:
            want = [x.clone() for x in (L.s_O, L.colscale, L.Y, L.what_int)]
        assert all(torch.equal(a, b) for a, b in zip(want, (L.s_O, L.colscale, L.Y, L.what_int)))


# the preparation's launch where every workgroup gathers the outlier columns itself: both sides of 2048 values, 512 rows and, without
# an adapter, 2048 and 12288 channels; one and 64 outliers, owners of rows alone and filled up, more channels than extra workgroups
_GATHERED = [(16, 3072, 4112, 31, 16), (512, 1040, 2064, 4, 16), (513, 1040, 2064, 3, 16), (32, 4112, 9232, 64, 16), (33, 4112, 1040, 64, 16),
             (1, 8192, 16384, 1, 16), (9, 2064, 2032, 5, 0), (9, 2064, 2048, 5, 0), (40, 2064, 12288, 33, 0), (40, 2064, 12272, 33, 0),
             (257, 2064, 528, 7, 16), (3, 7680, 528, 17, 0)]


@pytest.mark.parametrize("t,c_in,c_out,n,r", _GATHERED, ids=["%dx%dx%d_n%d_r%d" % c for c in _GATHERED])
def test_gathered_maxima(t, c_in, c_out, n, r):
    test_fwd_few(t, c_in, c_out, n, r)
