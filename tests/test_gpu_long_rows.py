"""Rows of many entries, summed a wave at a time: averages around the line where
the loop over a row changes (32), rows that end inside a chunk of staged entries
or go over several, in a V-cycle against lane groups and in whole solves."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg
from test_gpu_wave_rows import matrix

pytestmark = pytest.mark.gpu

CASES = [  # rows, couplings on either side, rows coupled to every third one
    (640, 15, []),
    (1281, 16, []),
    (2111, 17, [1000]),
    (1999, 60, []),
    (3000, 140, [0, 1500, 2999]),
    (65, 40, []),
]


@pytest.mark.parametrize("fp32", [False, True])
@pytest.mark.parametrize("case", range(len(CASES)))
def test_long_rows(case, fp32, monkeypatch):
    """Another order of up to 2000 roundings in a row: 1e-12 in double and 2e-5 in single precision of the largest
    entry, as for shorter rows (their errors grow with the root of the number)."""
    import torch

    n, width, hubs = CASES[case]
    print(n, width, hubs, fp32, flush=True)
    rng = np.random.default_rng(100 + case)
    a = matrix(n, list(range(1, width + 1)), hubs, rng)
    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    rh = rng.standard_normal(n)
    r = torch.from_numpy(rh).to("cuda:0")
    never = "2000000000"
    monkeypatch.setenv("HEMAMG_TAIL", "0")
    monkeypatch.setenv("HEMAMG_CODE_MIN", never)
    z = []
    for stream in (never, "1"):
        monkeypatch.setenv("HEMAMG_STREAM_MIN", stream)
        with hemamg.Hierarchy(A, precond_fp32=int(fp32), max_coarse_rows=16) as h:
            z.append(h.vcycle(r).cpu().numpy())
            for method in ("pcg", "bicgstab"):
                x, info = h.solve(r, rtol=1e-8, method=method)
                assert np.linalg.norm(rh - a.to_scipy() @ x.cpu().numpy()) <= 1.01e-8 * np.linalg.norm(rh)
    assert np.isfinite(z[0]).all()
    assert np.abs(z[1] - z[0]).max() <= (2e-5 if fp32 else 1e-12) * np.abs(z[0]).max()
