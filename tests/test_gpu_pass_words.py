"""The words by which a matching pass hands its sizes to the host, where other
read-backs of the same thread store values equal to the next sequence number."""
import threading

import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P
from test_gpu_parity import assert_same_hierarchy

pytestmark = pytest.mark.gpu


def stars_and_chain(stars, chain):
    """`stars` times 64 rows that never match (a row with eight stored zeros on either side of the diagonal of a
    symmetric pattern: nine distances, no edge), then a chain that halves in each pass."""
    n = 64 * stars + chain
    rows, cols, vals = [np.arange(n)], [np.arange(n)], [np.full(n, 4.0)]
    for g in range(stars):
        c, o = np.full(8, 64 * g), 64 * g + 1 + np.arange(8)
        rows += [c, o]
        cols += [o, c]
        vals += [np.zeros(8), np.zeros(8)]
    c = 64 * stars + np.arange(chain - 1)
    rows += [c, c + 1]
    cols += [c + 1, c]
    vals += [np.full(chain - 1, -1.0), np.full(chain - 1, -1.0)]
    r, c, v = (np.concatenate(t) for t in (rows, cols, vals))
    o = np.lexsort((c, r))
    rp = np.concatenate(([0], np.cumsum(np.bincount(r, minlength=n)))).astype(np.int32)
    return P.CSR(n, rp, c[o].astype(np.int32), v[o])


def uncoded(rp, ci):
    """Slices of 64 rows with more than 8 distances from the diagonal."""
    n, count = len(rp) - 1, 0
    for a in range(0, n, 64):
        b = min(a + 64, n)
        rows = np.repeat(np.arange(a, b), np.diff(rp[a:b + 1]))
        count += len(np.unique(ci[rp[a]:rp[b]] - rows)) > 8
    return count


def test_read_backs_leave_the_sequence_word(monkeypatch):
    """A setup ends with a read-back of its levels' slice counts.  Here level 11's is the number that the next
    setup's first pass waits for: a setup that finds it in the place of its sequence word takes stale sizes."""
    import torch

    assert torch.cuda.is_available()
    monkeypatch.setenv("HEMAMG_CODE_MIN", "1")
    monkeypatch.setenv("HEMAMG_MID_MIN", "1")
    # the chain's 4096 rows take 12 passes, a last one merges nothing: the next pass is the 14th
    a = stars_and_chain(stars=14, chain=4096)
    b = P.poisson3d(17, 13, 11)
    kw = dict(passes_per_level=1, max_coarse_rows=1, stall_ratio=1.0)
    failures = []

    def own_thread():  # a thread's words and its sequence numbers are its own
        try:
            A, B = hemamg.DeviceCSR.from_host(a, device="cuda:0"), hemamg.DeviceCSR.from_host(b, device="cuda:0")
            with hemamg.Hierarchy(A, **kw) as g, hemamg.Hierarchy(B) as h:
                rp, ci, _, _ = g.level(11)
                passes = len(g.stats()["rounds"])
                print("passes", passes, "slices without a code on level 11", uncoded(rp, ci), flush=True)
                assert uncoded(rp, ci) == passes + 1
                assert_same_hierarchy(g, oracle.Hierarchy(a, **kw))
                assert_same_hierarchy(h, oracle.Hierarchy(b))
        except BaseException as e:  # noqa: BLE001 (re-raised in the test's thread)
            failures.append(e)

    t = threading.Thread(target=own_thread)
    t.start()
    t.join()
    if failures:
        raise failures[0]


def test_refused_setup_returns_with_the_stream_finished():
    """A pattern that is not symmetric, found in the first pass of 343,000 rows: its sizes come from the first of
    many blocks, and the setup returns once they all have ended."""
    import torch

    a = P.poisson3d(70)
    keep = np.ones(len(a.col), bool)
    keep[a.row_ptr[1234] + 1] = a.col[a.row_ptr[1234] + 1] == 1234  # one entry of row 1234, not its mirror image
    assert keep.sum() == len(a.col) - 1
    rows = np.repeat(np.arange(a.n), np.diff(a.row_ptr))[keep]
    rp = np.concatenate(([0], np.cumsum(np.bincount(rows, minlength=a.n)))).astype(np.int32)
    A = hemamg.DeviceCSR.from_host(P.CSR(a.n, rp, a.col[keep], a.val[keep]), device="cuda:0")
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    for _ in range(20):
        with pytest.raises(hemamg.AmgError) as e:
            hemamg.Hierarchy(A, stream=s)
        assert s.query()
        assert e.value.status == hemamg.AMG_EINVAL
