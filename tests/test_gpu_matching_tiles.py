"""Matching passes in small tiles, for every form of the kernel: records of 4, 16
and 32 entries, in the workgroups of few and of many rows, with edges from tile
to tile in each, rows of more lower neighbours than a word holds, and stored
zeros.  Every hierarchy must be the oracle's, bit for bit."""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P
from test_gpu_parity import assert_same_hierarchy

pytestmark = pytest.mark.gpu


def symmetric(n, i, j, w):
    """The entries (i, j), i < j, and their mirror images, with a dominant diagonal; of equal pairs the first counts."""
    _, first = np.unique(i.astype(np.int64) * n + j, return_index=True)
    i, j, w = i[first], j[first], w[first]
    d = np.ones(n)
    np.add.at(d, i, np.abs(w))
    np.add.at(d, j, np.abs(w))
    r, c, v = np.concatenate((i, j, np.arange(n))), np.concatenate((j, i, np.arange(n))), np.concatenate((w, w, d))
    o = np.lexsort((c, r))
    rp = np.concatenate(([0], np.cumsum(np.bincount(r, minlength=n)))).astype(np.int32)
    return P.CSR(n, rp, c[o].astype(np.int32), v[o])


def band(n, width, reach, seed, zeros=0.0, hubs=()):
    """`width` couplings a row to rows up to `reach` further, integer weights with ties, a share of stored zeros, and
    every row coupled to each of the hubs."""
    rng = np.random.default_rng(seed)
    i = np.repeat(np.arange(n), width)
    j = i + rng.integers(1, reach + 1, len(i))
    i, j = i[j < n], j[j < n]
    for h in hubs:
        o = np.delete(np.arange(n), h)
        i, j = np.concatenate((i, np.minimum(o, h))), np.concatenate((j, np.maximum(o, h)))
    w = -rng.choice([1.0, 2.0, 3.0], len(i))
    w[rng.random(len(i)) < zeros] = 0.0
    return symmetric(n, i, j, w)


def form(n, nnz, n0, nnz0):
    """Record entries and threads a workgroup of a pass over n rows, of a setup of n0 rows."""
    avg = nnz / n
    rec = 4 if avg <= 7.5 else 16 if avg <= 14.0 else 32
    if rec == 32 and 32 * n > (32 if nnz0 > 14 * n0 else 16) * n0:
        rec = 16
    long_rows = rec == 32 and avg > 32.0  # tiles of 8 rows by themselves
    return rec, 512 if rec == 4 else 256 if n > 10000 or long_rows else 1024


CASES = {  # the matrix, and the forms its passes take
    "short rows": (lambda: band(1500, 3, 90, 1), {(4, 512)}),
    "short rows, stored zeros": (lambda: band(1500, 3, 90, 2, zeros=0.15), {(4, 512)}),
    "mid rows": (lambda: band(1500, 5, 200, 3, zeros=0.1), {(16, 1024)}),
    "mid rows, many": (lambda: band(12007, 5, 300, 4), {(16, 256)}),
    "long rows": (lambda: band(1500, 16, 300, 5, zeros=0.1), {(32, 1024)}),
    "long rows, many": (lambda: band(42011, 14, 500, 6, zeros=0.05), {(32, 256)}),
    "very long rows": (lambda: band(1300, 40, 400, 8, zeros=0.1, hubs=(700,)), {(32, 256)}),
    "hubs": (lambda: band(1500, 3, 60, 7, zeros=0.1, hubs=(0, 400, 1100, 1499)), {(32, 1024)}),
}


@pytest.mark.parametrize("alternate", [0, 1])
@pytest.mark.parametrize("tile", [0, 1, 37, 64, 101])
@pytest.mark.parametrize("name", list(CASES))
def test_small_tiles(name, tile, alternate, monkeypatch):
    print("case", name, "tile", tile, alternate, flush=True)
    monkeypatch.setenv("HEMAMG_HEM_TILE", str(tile))
    make, forms = CASES[name]
    a = make()
    with hemamg.Hierarchy(hemamg.DeviceCSR.from_host(a, device="cuda:0"), alternate=alternate) as g:
        s = g.stats()
        assert forms <= {form(n, z, a.n, a.nnz) for n, z in zip(s["pass_n"], s["pass_nnz"])}
        assert_same_hierarchy(g, oracle.Hierarchy(a, alternate=alternate))
