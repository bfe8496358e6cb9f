"""bench.py's byte counts follow the kernels that the levels of a hierarchy run."""
import os
import sys

import numpy as np
import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
if ROOT not in sys.path:
    sys.path.insert(0, ROOT)

import bench  # noqa: E402
from paper_2007_00056_amd import problems as P  # noqa: E402


def test_slices_fit():
    a = P.poisson3d(20, 17, 13)
    assert bench.slices_fit(a.row_ptr, a.col)
    r = P.random_symmetric_pattern(3000, 0.003, 1)
    assert not bench.slices_fit(r.row_ptr, r.col)
    # a slice without a code is spared at 64 slices, not below
    for n, ok in ((64 * 64, True), (64 * 63, False)):
        far = np.arange(9, 18) * 64
        rows, cols = np.concatenate((np.arange(n), np.arange(9))), np.concatenate((np.arange(n), far))
        o = np.lexsort((cols, rows))
        rp = np.concatenate(([0], np.cumsum(np.bincount(rows, minlength=n))))
        assert bench.slices_fit(rp, cols[o]) is ok


@pytest.mark.parametrize("e", [8, 4])
def test_levels_with_codes_read_no_columns(e):
    """128^3 and its first coarse levels, all of the grid's pattern, in single precision coded above 262,144 rows only."""
    sizes = [(128 ** 3 // 4 ** k, 7 * 128 ** 3 // 4 ** k) for k in range(6)]
    grid = P.poisson3d(16)
    kinds = bench.row_kinds(sizes, e, lambda k: (grid.row_ptr, grid.col))
    assert [c for c, _ in kinds] == [True, True, e == 8, False, False]
    assert [k for _, k in kinds] == ["coded", "coded", "coded" if e == 8 else "stream", "group", "group"]
    for k in range(5):
        n, nnz = sizes[k]
        if kinds[k][0]:  # both directions: 4 bytes an entry and 2 a row less
            assert (bench.level_bytes(k, sizes, e, "stream") - bench.level_bytes(k, sizes, e, "coded")
                    == 2 * (4 * nnz + 4 * (n + 1) - 2 * n))
    every = bench.iteration_bytes(sizes, "pcg", e, kinds)
    first = bench.iteration_bytes(sizes, "pcg", e, [kinds[0]] + [(False, "stream" if k == "coded" else k) for _, k in kinds[1:]])
    coded = [sizes[k] for k in range(1, 5) if kinds[k][0]]
    assert first - every == sum(2 * (4 * nnz + 4 * (n + 1) - 2 * n) for n, nnz in coded)


def test_small_level_0_keeps_lane_groups_in_the_cycle():
    a = P.poisson2d(64)
    kinds = bench.row_kinds([(a.n, a.nnz), (1024, 5000), (64, 300)], 8, lambda k: (a.row_ptr, a.col))
    assert kinds[0] == (True, "group")  # the outer products read codes
    long_rows = bench.row_kinds([(100000, 5000000), (30000, 900000)], 8, lambda k: None)
    assert long_rows == [(False, "group")]
