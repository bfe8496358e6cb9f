"""Matching kernel at the sizes where its forms change: record lengths (4, 16
and 32 higher neighbours), more lower neighbours than a word holds, and tile
boundaries.  Every hierarchy must be the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def same_hierarchy(a, **kw):
    import torch

    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    o = oracle.Hierarchy(a, **kw)
    with hemamg.Hierarchy(A, **kw) as g:
        torch.cuda.synchronize()
        assert g.nlevels == o.nlevels
        for k in range(o.nlevels):
            rp, ci, v, agg = g.level(k)
            ol = o.level(k)
            np.testing.assert_array_equal(rp, ol.row_ptr)
            np.testing.assert_array_equal(ci, ol.col)
            np.testing.assert_array_equal(v.view(np.int64), ol.val.view(np.int64))
            if ol.agg is not None:
                np.testing.assert_array_equal(agg, ol.agg)


def banded(n, width, seed):
    """Every row coupled to `width` rows on either side, random integer weights with ties."""
    rng = np.random.default_rng(seed)
    a = np.zeros((n, n))
    for d in range(1, width + 1):
        w = -rng.choice([1.0, 2.0, 3.0], size=n - d)
        a[np.arange(n - d), np.arange(d, n)] = w
        a[np.arange(d, n), np.arange(n - d)] = w
    np.fill_diagonal(a, np.abs(a).sum(axis=1) + 1.0)
    return P.from_dense(a)


@pytest.mark.parametrize("alternate", [0, 1])
@pytest.mark.parametrize("width", [3, 4, 5, 15, 16, 17, 30, 31, 32, 33, 70])
def test_list_lengths(width, alternate):
    """`width` higher and lower neighbours each: records end, go on in the row, and the
    lower edges fill a word (31), or need further ones."""
    print("width", width, flush=True)
    same_hierarchy(banded(300, width, width), max_coarse_rows=16, alternate=alternate)


@pytest.mark.parametrize("n", [1, 2, 127, 128, 129, 383, 384, 385, 895, 896, 897, 10001])
@pytest.mark.parametrize("width", [2, 6])
def test_tile_edges(n, width):
    """Chains with `width` neighbours a side around the tile sizes (128, 384 and 896 rows, and where the
    large tiles end)."""
    print("n", n, "width", width, flush=True)
    rng = np.random.default_rng(n)
    off = [d for d in range(1, width + 1) if d < n]
    rows, cols, vals = [np.arange(n)], [np.arange(n)], [np.full(n, 100.0)]
    for d in off:
        w = -rng.choice([1.0, 2.0, 3.0], size=n - d)
        rows += [np.arange(n - d), np.arange(d, n)]
        cols += [np.arange(d, n), np.arange(n - d)]
        vals += [w, w]
    r, c, v = (np.concatenate(t) for t in (rows, cols, vals))
    o = np.lexsort((c, r))
    rp = np.concatenate(([0], np.cumsum(np.bincount(r, minlength=n)))).astype(np.int32)
    same_hierarchy(P.CSR(n, rp, c[o].astype(np.int32), v[o]), max_coarse_rows=1 if n < 3 else 64)


@pytest.mark.parametrize("hub", ["first", "middle", "last"])
def test_long_rows(hub):
    """A row coupled to every other one, its neighbours also in a chain: a list and a set of lower edges
    far beyond a record and a word, with stored zeros among them."""
    n = 1200
    h = {"first": 0, "middle": n // 2, "last": n - 1}[hub]
    rng = np.random.default_rng(5)
    a = np.zeros((n, n))
    mask = np.eye(n, dtype=bool)
    for d in (1, 2):
        w = -rng.choice([1.0, 2.0], size=n - d)
        a[np.arange(n - d), np.arange(d, n)] = w
        a[np.arange(d, n), np.arange(n - d)] = w
    w = -rng.choice([0.0, 1.0, 2.0, 3.0], size=n)
    a[h, :] = w
    a[:, h] = w
    mask[h, :] = mask[:, h] = True
    np.fill_diagonal(a, np.abs(a).sum(axis=1) + 1.0)
    mask |= a != 0
    r, c = np.nonzero(mask)
    rp = np.concatenate(([0], np.cumsum(np.bincount(r, minlength=n)))).astype(np.int32)
    same_hierarchy(P.CSR(n, rp, c.astype(np.int32), a[r, c]))
