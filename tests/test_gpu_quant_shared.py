"""The stand-alone quantizer where four rows share their column scales: both sides of its limits (3072 and 4096 columns at any number of
rows, 2048 rows without outliers, 6144 and 1920 to 2048 or 2400 with them, 128 outliers), ragged rows, rows that end inside a wavefront, a leading dimension of its own, a zero row,
no and many outliers, against the oracle: codes, steps and compact outlier codes bit for bit."""
import sys

import numpy as np
import pytest

pytestmark = pytest.mark.gpu

# (t, c, number of outliers, padding of a row)
_CASES = [(1, 3088, 0, 0), (7, 4096, 128, 8), (258, 3584, 5, 0), (130, 4112, 3, 0), (2047, 4112, 0, 0), (2049, 4112, 0, 16), (2050, 8208, 65, 0),
          (2047, 8208, 1, 0), (4097, 4112, 40, 0), (4095, 4112, 40, 0), (2051, 16384, 129, 0), (2051, 16384, 128, 0), (2048, 12288, 0, 0)]

# the limits with outliers: 6144 rows up to 4096 columns and from 6145 on, 11264 columns, 1920 to 2048 and from 2400 rows beyond
_CASES += [(6143, 4096, 3, 0), (6145, 4096, 3, 0), (6145, 6144, 5, 0), (6145, 6160, 5, 8), (6143, 6160, 128, 0), (2401, 11264, 9, 0),
           (2401, 11280, 9, 0), (2399, 11280, 9, 0), (2049, 11280, 9, 0), (2047, 11280, 9, 0), (1919, 11280, 9, 0)]


@pytest.mark.parametrize("t,c,n,pad", _CASES, ids=["%dx%d_n%d_pad%d" % x for x in _CASES])
def test_quant_shared(t, c, n, pad):
    import torch
    from oracle import api as orc
    from paper_2505_14742_amd import binding as q
    from tests.gpu_harness import DEV, bf16_dev, dev, host
    print("quant shared", t, c, n, pad, flush=True)
    sys.stdout.flush()
    rng = np.random.default_rng(t + c + n)
    X = (rng.standard_normal((t, c), dtype=np.float32).view(np.uint32) >> 16).astype(np.uint16)
    X[t // 2] = 0
    O = np.sort(rng.permutation(c)[:n]).astype(np.int32)
    cs = np.ones(c, np.float32)
    cs[O] = rng.uniform(0.01, 1.0, n).astype(np.float32)
    if n:
        O[0], O[-1] = (0, c - 1) if n > 1 else (c - 1, c - 1)
    wide = np.zeros((t, c + pad), np.uint16)
    wide[:, :c] = X
    Xd = bf16_dev(wide)[:, :c]
    n_pad = q.padded_outliers(n)
    Xq = torch.full((t, c), 77, dtype=torch.int8, device=DEV)
    delta = torch.full((t,), -1.0, device=DEV)
    xo = torch.full((t, n_pad), 55, dtype=torch.int8, device=DEV) if n else None
    q.quant_act(Xd, dev(cs), dev(O) if n else None, Xq, delta, xo)
    want, d, x = orc.quant_act(X, cs, O)
    assert np.array_equal(host(Xq), want) and np.array_equal(host(delta), d)
    if n:
        assert np.array_equal(host(xo)[:, :n], x) and not host(xo)[:, n:].any()
