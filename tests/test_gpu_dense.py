"""Coarsest inverse at the sizes where its kernels change (one workgroup up to
64 and 128 rows; panels of 16 columns with 1 or 2 rows a thread, of 8 with 4),
on matrices whose pivots are off the diagonal."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def dense_csr(a):
    n = a.shape[0]
    return P.CSR(n, np.arange(0, n * n + 1, n, dtype=np.int32), np.tile(np.arange(n, dtype=np.int32), n),
                 np.ascontiguousarray(a).reshape(-1))


@pytest.mark.parametrize("n", [1, 2, 15, 63, 64, 65, 127, 128, 129, 144, 256, 257, 513, 1024, 1025, 2049])
def test_single_level_solve(n):
    """max_coarse_rows = n: one V-cycle is the exact solve.  Rows of a diagonally dominant matrix in random
    order (condition number below 10, no zero on the diagonal): the error stays within 1e-11, n times the
    rounding unit with room for the condition number and the explicit inverse."""
    import torch

    print("n", n, flush=True)
    rng = np.random.default_rng(n)
    a = rng.uniform(0.1, 1.0, (n, n)) * rng.choice([-1.0, 1.0], (n, n)) * (1.0 / n)
    a[np.arange(n), rng.permutation(n)] += 2.0
    A = hemamg.DeviceCSR.from_host(dense_csr(a), device="cuda:0")
    b = rng.uniform(-1.0, 1.0, n)
    with hemamg.Hierarchy(A, max_coarse_rows=n) as h:
        assert h.nlevels == 1
        x = h.vcycle(torch.from_numpy(b).to("cuda:0")).cpu().numpy()
    ref = np.linalg.solve(a, b)
    assert np.linalg.norm(x - ref) <= 1e-11 * np.linalg.norm(ref)
    assert np.abs(x - ref).max() <= 1e-11 * np.abs(ref).max()


@pytest.mark.parametrize("n", [2, 40, 100, 200])
def test_singular(n):
    """Rank n - 1 with exact arithmetic (two equal rows of small integers in a permuted identity): rejected."""
    a = np.eye(n) * 2.0
    a[0, 1] = a[1, 0] = 2.0
    A = hemamg.DeviceCSR.from_host(dense_csr(a), device="cuda:0")
    with pytest.raises(hemamg.AmgError) as e:
        hemamg.Hierarchy(A, max_coarse_rows=n)
    assert e.value.status == hemamg.AMG_ESINGULAR
