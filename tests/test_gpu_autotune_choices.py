"""The autotuner leaves alone what has no choice: small levels that run in one
workgroup, and the rows per block of levels whose columns are coded."""
import numpy as np
import pytest

from paper_2007_00056_amd import hemamg, problems as P

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("fp32", [0, 1])
def test_levels_without_a_choice(fp32):
    import torch

    a = P.poisson3d(40)  # 64,000 rows with codes; the levels below 1000 rows in one workgroup
    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    b = torch.from_numpy(P.rhs_uniform(a.n, 1)).to("cuda:0")
    with hemamg.Hierarchy(A, precond_fp32=fp32) as g:
        sizes = [hemamg.amg_level_size(g.h, k)[0] for k in range(g.nlevels)]
        x0, i0 = g.solve(b)
        for _ in range(4):
            sched = g.autotune()
            print(sizes, sched, flush=True)
            assert sched[0] in (256, -2, -4, -8) and sched[-1] == 0
            assert [s for n, s in zip(sizes[:-1], sched) if n < 300] == [256] * sum(n < 300 for n in sizes[:-1])
        x1, i1 = g.solve(b)
        assert abs(i0["iters"] - i1["iters"]) <= 1
        assert (x0 - x1).abs().max().item() <= 1e-6 * x0.abs().max().item()


def test_coded_level_of_a_batch():
    import torch

    systems = [P.poisson3d(16), P.poisson3d(20, 17, 11)]
    devs = [hemamg.DeviceCSR.from_host(a, device="cuda:0") for a in systems]
    rhs = torch.from_numpy(np.concatenate([P.rhs_uniform(a.n, k) for k, a in enumerate(systems)])).to("cuda:0")
    bt = hemamg.Batch.setup(devs, hemamg.amg_params_default())
    try:
        x0, _ = bt.solve(rhs, rtol=1e-8)
        for _ in range(4):
            sched = bt.autotune()
            assert sched[0] == 256 and sched[-1] == 0
        x1, _ = bt.solve(rhs, rtol=1e-8)
        assert torch.equal(x0, x1)
    finally:
        bt.close()
