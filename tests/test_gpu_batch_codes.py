"""A batch's level 0 read through column codes against its CSR rows: the same
iterates bit for bit, with system borders inside slices of 64 rows."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def grid(nx, ny, rng):
    import scipy.sparse as sp

    n = nx * ny
    e = rng.uniform(0.5, 1.5, n) * (np.arange(n) % nx != nx - 1)
    s = rng.uniform(0.5, 1.5, n - nx)
    u = sp.diags(-e[:-1], 1, shape=(n, n)) + sp.diags(-s, nx, shape=(n, n))
    u = u.tocsr()
    u.eliminate_zeros()
    a = (u + u.T).tocsr()
    a = (a + sp.diags(np.asarray(abs(a).sum(1)).ravel() + 0.02)).tocsr()
    a.sort_indices()
    return P.CSR(n, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64))


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("sides", [[(80, 79), (61, 103), (97, 66)], [(90, 71)], [(9, 8)] * 70])
def test_same_bits(sides, fp32, monkeypatch):
    """The last batch has a border in almost every slice: no codes, the CSR rows as before."""
    import torch

    print(sides[:3], len(sides), fp32, flush=True)
    rng = np.random.default_rng(len(sides))
    A = [hemamg.DeviceCSR.from_host(grid(*s, rng), device="cuda:0") for s in sides]
    b = torch.from_numpy(rng.standard_normal(sum(x * y for x, y in sides))).to("cuda:0")
    out = []
    for code_min in ("1", "2000000000"):
        monkeypatch.setenv("HEMAMG_CODE_MIN", code_min)
        for method in ("pcg", "bicgstab"):
            with hemamg.Batch.setup(A, precond_fp32=fp32, max_coarse_rows=20) as bt:
                x, info = bt.solve(b, rtol=1e-8, method=method)
                assert all(i["status"] == hemamg.AMG_OK for i in info)
                out.append(x.cpu().numpy())
    assert np.array_equal(out[0], out[2]) and np.array_equal(out[1], out[3])
