"""The way down that forms D^{-1} r itself on level 0 (a V-cycle on a caller's
vector) against the one that is handed it (inside CG): the first direction of a
CG solve is that V-cycle, so one iteration must give x along it; in every kind
of level-0 kernel."""
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
    return P.CSR(n, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64)), a


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("n,bands", [(65, [1]), (1000, [1, 10]), (3001, [1, 14, 200]), (2000, list(range(1, 9)))])
@pytest.mark.parametrize("mid,code", [("2000000000", "2000000000"), ("1", "2000000000"), ("1", "1")])
def test_first_direction(n, bands, mid, code, fp32, monkeypatch):
    """x = alpha z with alpha = (b, z) / (z, A z): a few roundings of sums over n terms, 1e-11 relative."""
    import torch

    print(n, bands[:3], mid, code, fp32, flush=True)
    monkeypatch.setenv("HEMAMG_MID_MIN", mid)
    monkeypatch.setenv("HEMAMG_CODE_MIN", code)
    rng = np.random.default_rng(n)
    a, m = laplacian(n, bands, rng)
    b = rng.standard_normal(n)
    d = torch.from_numpy(b).to("cuda:0")
    with hemamg.Hierarchy(hemamg.DeviceCSR.from_host(a, device="cuda:0"), precond_fp32=fp32, max_coarse_rows=16) as h:
        z = h.vcycle(d).cpu().numpy()
        x = h.solve(d, rtol=1e-14, maxit=1, check=False)[0].cpu().numpy()
    want = (b @ z) / (z @ (m @ z)) * z
    assert np.abs(x - want).max() <= 1e-11 * np.abs(want).max()
