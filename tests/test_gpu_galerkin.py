"""Galerkin product at the row lengths where its kernels change: entries of a
coarse row around one and two a lane, for 16 and for 32 lanes a row, and above
(the slow path), with many and with few equal coarse columns.  Every hierarchy
must be the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def pairs(n, band, entries, near, rng):
    """Strongly coupled pairs (2i, 2i + 1), weak couplings to `band` rows on either side of a pair, and three pairs
    whose rows have `entries` entries together, to near or to far columns."""
    a = np.zeros((n, n))

    def couple(i, j, w):
        if i != j:
            a[i, j] = a[j, i] = -w

    for d in range(2, band + 2):
        for i in range(n - d):
            couple(i, i + d, rng.uniform(0.01, 0.1))
    for i in range(0, n - 1, 2):
        couple(i, i + 1, 10.0 + rng.uniform(0.0, 1.0))
    for i in (100, 250, 400):
        have = np.count_nonzero(a[i]) + np.count_nonzero(a[i + 1]) + 2
        free = [j for j in (range(i + 2, n) if near else rng.permutation(n)) if a[i, j] == 0.0 and j not in (i, i + 1)]
        for j in free[: max(0, entries - have)]:
            couple(i, j, rng.uniform(0.001, 0.01))
    np.fill_diagonal(a, np.abs(a).sum(axis=1) + 1.0)
    return P.from_dense(a)


@pytest.mark.parametrize("near", [False, True])
@pytest.mark.parametrize("band,entries", [(0, 15), (0, 16), (0, 17), (0, 31), (0, 32), (0, 33), (0, 200),
                                          (6, 31), (6, 32), (6, 33), (6, 63), (6, 64), (6, 65), (6, 300)])
def test_row_lengths(band, entries, near):
    import torch

    print(band, entries, near, flush=True)
    a = pairs(600, band, entries, near, np.random.default_rng(entries))
    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    o = oracle.Hierarchy(a, max_coarse_rows=20)
    with hemamg.Hierarchy(A, max_coarse_rows=20) as g:
        torch.cuda.synchronize()
        assert g.nlevels == o.nlevels
        for k in range(o.nlevels):
            rp, ci, v, _ = g.level(k)
            ol = o.level(k)
            np.testing.assert_array_equal(rp, ol.row_ptr)
            np.testing.assert_array_equal(ci, ol.col)
            np.testing.assert_array_equal(v.view(np.int64), ol.val.view(np.int64))
