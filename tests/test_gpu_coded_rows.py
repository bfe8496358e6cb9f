"""Level-0 rows read through per-slice column codes against the same rows read
from the CSR arrays: a V-cycle and whole solves agree bit for bit, since both
add a row's products in entry order."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def stencil(n, offsets, rng, keep=1.0, extra=()):
    """Diagonally dominant symmetric matrix with entries at the offsets (each kept with probability keep)
    and at the extra (row, col) pairs."""
    import scipy.sparse as sp

    a = sp.lil_matrix((n, n)) if extra else None
    parts = []
    for d in offsets:
        if d < n:
            v = -rng.uniform(0.5, 1.5, n - d) * (rng.random(n - d) < keep)
            parts.append(sp.coo_matrix((v, (np.arange(n - d), np.arange(d, n))), shape=(n, n)))
    if extra:
        for i, j in extra:
            a[min(i, j), max(i, j)] = -0.1
        parts.append(a.tocoo())
    u = sum(p.tocsr() for p in parts)
    u.eliminate_zeros()
    a = (u + u.T).tocsr()
    a = a + sp.diags(np.asarray(abs(a).sum(1)).ravel() + 0.05)
    a = a.tocsr()
    a.sort_indices()
    return P.CSR(n, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64))


def cases():
    rng = np.random.default_rng(7)
    yield "tridiagonal, n = 64 k", stencil(640, [1], rng)
    yield "5 distances, n = 64 k + 1", stencil(1345, [1, 37], rng)
    yield "7 distances, n = 64 k - 1", stencil(4991, [1, 17, 290], rng)
    yield "7 distances, a third of the entries missing", stencil(7003, [1, 19, 333], rng, keep=0.67)
    yield "a slice with couplings of its own", stencil(6500, [1, 20, 400], rng, extra=[(3200 + k, 3200) for k in (2, 3, 5, 7)])
    yield "the last slice with couplings of its own", stencil(6465, [1, 20, 400], rng,
                                                              extra=[(6464, 6464 - k) for k in range(2, 15)])
    yield "no slice fits", stencil(3000, [1], rng,
                                   extra=[(k, k * 7919 % 3000) for k in range(0, 3000, 2) if k != k * 7919 % 3000])


CASES = list(cases())


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)), ids=[c[0] for c in CASES])
def test_coded_rows_equal_csr_rows(case, fp32, monkeypatch):
    import torch

    name, A = CASES[case]
    print(name, A.n, fp32, flush=True)
    rng = np.random.default_rng(case)
    b = torch.from_numpy(rng.standard_normal(A.n)).to("cuda:0")
    dev = hemamg.DeviceCSR.from_host(A, device="cuda:0")
    monkeypatch.setenv("HEMAMG_STREAM_MIN", "1")
    out = []
    for code_min in ("1", "2000000000"):
        monkeypatch.setenv("HEMAMG_CODE_MIN", code_min)
        with hemamg.Hierarchy(dev, precond_fp32=fp32) as h:
            res = [h.vcycle(b)]
            for method in ("pcg", "bicgstab"):
                res.append(h.solve(b, method=method, rtol=1e-9)[0])
            out.append([r.cpu().numpy() for r in res])
    for coded, csr in zip(*out):
        assert np.isfinite(csr).all()
        assert np.array_equal(coded, csr)
