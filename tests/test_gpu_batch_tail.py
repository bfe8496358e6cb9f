"""Batched solves whose small levels run in one workgroup per system against the
same levels in kernels for the whole batch: the same iterates bit for bit, with
systems whose levels fit from level 1 on, from a later one, or not at all."""
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


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("coarse", [20, 140, 300])
def test_same_bits(fp32, coarse, monkeypatch):
    """coarse: rows below which a system is solved directly; above 256 no system has a tail."""
    import torch

    print(fp32, coarse, flush=True)
    rng = np.random.default_rng(coarse)
    mats = [laplacian(n, b, rng) for n, b in
            [(700, [1]), (1900, [1, 40]), (5000, [1, 17, 290]), (20000, [1, 27, 729]), (310, list(range(1, 20)))]]
    A = [hemamg.DeviceCSR.from_host(m, device="cuda:0") for m in mats]
    b = torch.from_numpy(rng.standard_normal(sum(m.n for m in mats))).to("cuda:0")
    par = hemamg.amg_params_default(precond_fp32=fp32, max_coarse_rows=coarse)
    out = {}
    for lds in ("0", "1000000"):
        monkeypatch.setenv("HEMAMG_TAIL", lds)
        for method in ("pcg", "bicgstab"):
            with hemamg.Batch.setup(A, params=par) as bt:
                x, info = bt.solve(b, rtol=1e-8, method=method)
                out[lds, method] = x.cpu().numpy()
                assert all(i["status"] == hemamg.AMG_OK for i in info)
            hs = [hemamg.Hierarchy(a, params=par) for a in A]
            with hemamg.Batch(hs) as bt:
                x, _ = bt.solve(b, rtol=1e-8, method=method)
                assert np.array_equal(x.cpu().numpy(), out[lds, method])
            for h in hs:
                h.close()
    for method in ("pcg", "bicgstab"):
        assert np.array_equal(out["0", method], out["1000000", method])
