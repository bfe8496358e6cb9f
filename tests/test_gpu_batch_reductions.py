"""Batched CG adds a system's block partials in the kernels that use them, up to
512 blocks of 256 rows; with a larger system in the batch a kernel of its own
does.  A small system's iterates are the same bit for bit in either batch."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


def path(n, rng):
    w = rng.uniform(0.5, 1.5, n - 1)
    rows = np.concatenate([np.arange(n), np.arange(n - 1), np.arange(1, n)])
    cols = np.concatenate([np.arange(n), np.arange(1, n), np.arange(n - 1)])
    vals = np.concatenate([0.2 + np.append(w, 0.0) + np.append(0.0, w), -w, -w])
    order = np.lexsort((cols, rows))
    rp = np.concatenate([[0], np.cumsum(np.bincount(rows, minlength=n))]).astype(np.int32)
    return P.CSR(n, rp, cols[order].astype(np.int32), np.ascontiguousarray(vals[order]))


@pytest.mark.parametrize("fp32", [0, 1])
@pytest.mark.parametrize("large", [512 * 256, 512 * 256 + 1])
def test_small_system_beside_a_large_one(large, fp32):
    import torch

    print(large, fp32, flush=True)
    rng = np.random.default_rng(3)
    mats = [path(n, rng) for n in (255, 257, 5000, large)]
    A = [hemamg.DeviceCSR.from_host(m, device="cuda:0") for m in mats]
    b = torch.from_numpy(rng.standard_normal(sum(m.n for m in mats))).to("cuda:0")
    few = 255 + 257 + 5000
    out = []
    for k, rhs in ((3, b[:few].clone()), (4, b)):
        with hemamg.Batch.setup(A[:k], precond_fp32=fp32) as bt:
            x, info = bt.solve(rhs, rtol=1e-9)
            assert all(i["status"] == hemamg.AMG_OK and i["true_rel_res"] <= 2e-9 for i in info)
            out.append(x[:few].cpu().numpy())
    assert np.array_equal(out[0], out[1])
