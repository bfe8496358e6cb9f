"""CSR rows summed a wave at a time: in the lane-group kernels' order the cycle
is theirs bit for bit, in entry order it is within rounding; with row counts
around 64, rows longer than a wave's chunk of entries, and chunks that end
inside a row."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def matrix(n, bands, hubs, rng):
    """Band matrix with `hubs` rows (and columns) coupled to every third row."""
    import scipy.sparse as sp

    u = sum(sp.diags(-rng.uniform(0.5, 1.5, n - d), d, shape=(n, n)) for d in bands if d < n).tocsr()
    if hubs:
        far = np.array([(h, j) for h in hubs for j in range(0, n, 3) if abs(h - j) > max(bands) and j not in hubs])
        far.sort(axis=1)
        u = u + sp.coo_matrix((-rng.uniform(0.01, 0.02, len(far)), (far[:, 0], far[:, 1])), shape=(n, n)).tocsr()
    a = (u + u.T).tocsr()
    a = (a + sp.diags(np.asarray(abs(a).sum(1)).ravel() + 0.02)).tocsr()
    a.sort_indices()
    return P.CSR(n, a.indptr.astype(np.int32), a.indices.astype(np.int32), a.data.astype(np.float64))


CASES = [
    (63, [1], []),
    (640, [1, 20], []),
    (2113, [1, 7, 49], [5]),
    (1999, list(range(1, 9)), []),
    (1500, list(range(1, 25)), [0, 700]),
    (9001, [1, 90], [64, 8999]),
]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_wave_rows(case, fp32, monkeypatch):
    """Entry order against lane groups: another order of a few hundred roundings, 1e-12 in double and 2e-5 in
    single precision of the largest entry."""
    import torch

    n, bands, hubs = CASES[case]
    print(n, bands[:4], hubs, fp32, flush=True)
    rng = np.random.default_rng(case)
    A = hemamg.DeviceCSR.from_host(matrix(n, bands, hubs, rng), device="cuda:0")
    r = torch.from_numpy(rng.standard_normal(n)).to("cuda:0")
    never = "2000000000"
    monkeypatch.setenv("HEMAMG_TAIL", "0")
    monkeypatch.setenv("HEMAMG_CODE_MIN", never)
    z = {}
    for name, stream, mid in (("groups", never, never), ("same order", never, "1"), ("entry order", "1", "1")):
        monkeypatch.setenv("HEMAMG_STREAM_MIN", stream)
        monkeypatch.setenv("HEMAMG_MID_MIN", mid)
        with hemamg.Hierarchy(A, precond_fp32=int(fp32), max_coarse_rows=16) as h:
            z[name] = h.vcycle(r).cpu().numpy()
            x, info = h.solve(r, rtol=1e-8)
            assert info["true_rel_res"] <= 2e-8
    assert np.isfinite(z["groups"]).all()
    assert np.array_equal(z["same order"], z["groups"])
    assert np.abs(z["entry order"] - z["groups"]).max() <= (2e-5 if fp32 else 1e-12) * np.abs(z["groups"]).max()
