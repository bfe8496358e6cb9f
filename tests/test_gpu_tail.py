"""The small levels of the V-cycle in one workgroup against the same levels in
kernels of their own: sizes around the kernel's edges (rows per step, lanes per
row, rows of the coarsest solve held in registers), one and two matching passes
a level, long rows."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def laplacian(n, bands, rng):
    import scipy.sparse as sp

    u = sum(sp.diags(-rng.uniform(0.5, 1.5, n - d), d, shape=(n, n)) for d in bands if d < n)
    a = (u + u.T).tocsr()
    a = (a + sp.diags(np.asarray(abs(a).sum(1)).ravel() + 0.02)).tocsr()
    a.sort_indices()
    return P.CSR(n, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64))


# rows, distances of the off-diagonals, options
CASES = [
    (40, [1], dict(max_coarse_rows=1)),
    (255, [1], dict(max_coarse_rows=16)),
    (257, [1, 9], dict(max_coarse_rows=65)),
    (1021, [1, 31], dict(max_coarse_rows=64)),
    (1030, [1], dict(max_coarse_rows=127)),
    (2050, [1, 40], dict(max_coarse_rows=130)),
    (4100, [1, 2], dict(max_coarse_rows=256)),
    (4400, [1], dict(max_coarse_rows=300)),
    (5800, [1], dict(max_coarse_rows=20)),
    (3000, [1], dict(max_coarse_rows=20, passes_per_level=1)),
    (1500, [1, 5, 25, 125], dict(max_coarse_rows=32, passes_per_level=1)),
    (1200, list(range(1, 30)), dict(max_coarse_rows=24)),
    (13000, [1, 23, 529], dict()),
]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_tail_matches_level_kernels(case, fp32, monkeypatch):
    """Both add the same terms in another order: a few hundred roundings deep in all, so 1e-12 in double and
    2e-5 in single precision, relative to the largest entry."""
    import torch

    n, bands, opt = CASES[case]
    print(n, bands[:4], opt, fp32, flush=True)
    rng = np.random.default_rng(case)
    A = hemamg.DeviceCSR.from_host(laplacian(n, bands, rng), device="cuda:0")
    r = torch.from_numpy(rng.standard_normal(n)).to("cuda:0")
    z = []
    for lds in ("0", "1000000"):
        monkeypatch.setenv("HEMAMG_TAIL", lds)
        with hemamg.Hierarchy(A, precond_fp32=int(fp32), **opt) as h:
            first = h.vcycle(r)
            again = h.vcycle(r)
            assert torch.equal(first, again)
            z.append(first.cpu().numpy())
    assert np.isfinite(z[0]).all()
    assert np.abs(z[1] - z[0]).max() <= (2e-5 if fp32 else 1e-12) * np.abs(z[0]).max()
