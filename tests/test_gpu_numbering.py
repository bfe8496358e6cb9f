"""Numbering and row offsets of a pass at the row counts where their prefix
sums change form (one workgroup up to 4096 and 16384 rows, tiles of 2048 above):
the hierarchy must be the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", [1, 5, 4095, 4096, 4097, 8200, 16383, 16384, 16385, 34817])
def test_sizes(n):
    import torch

    print("n", n, flush=True)
    rng = np.random.default_rng(n)
    w = rng.uniform(0.5, 1.5, max(n - 1, 0)) * (rng.random(max(n - 1, 0)) < 0.9)  # some rows alone
    rows = np.concatenate([np.arange(n), np.nonzero(w)[0], np.nonzero(w)[0] + 1])
    cols = np.concatenate([np.arange(n), np.nonzero(w)[0] + 1, np.nonzero(w)[0]])
    diag = 0.1 + np.concatenate([w, [0.0]])[:n] + np.concatenate([[0.0], w])[:n]
    vals = np.concatenate([diag, -w[w > 0], -w[w > 0]])
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    a = P.CSR(n, rp, cols[order].astype(np.int32), np.ascontiguousarray(vals[order]))
    opt = dict(max_coarse_rows=min(500, max(1, n // 3)), passes_per_level=1)
    o = oracle.Hierarchy(a, **opt) if n > 1 else None
    with hemamg.Hierarchy(hemamg.DeviceCSR.from_host(a, device="cuda:0"), **opt) as g:
        torch.cuda.synchronize()
        assert g.nlevels == (o.nlevels if o else 1)
        for k in range(g.nlevels if o else 0):
            rp, ci, v, agg = g.level(k)
            ol = o.level(k)
            np.testing.assert_array_equal(rp, ol.row_ptr)
            np.testing.assert_array_equal(ci, ol.col)
            np.testing.assert_array_equal(v.view(np.int64), ol.val.view(np.int64))
            if ol.agg is not None:
                np.testing.assert_array_equal(agg, ol.agg)
