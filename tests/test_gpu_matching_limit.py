"""Time limit of a matching pass: a pass that is given up ends, its repeat gives
the oracle's hierarchy, and the limit lies above what a long chain needs."""
import numpy as np
import pytest

import oracle
from paper_2007_00056_amd import hemamg, problems as P
from test_gpu_parity import assert_same_hierarchy

pytestmark = pytest.mark.gpu


def chain(n):
    """Tridiagonal: vertex 2k can decide once 2k - 2 has, one after the other."""
    i = np.arange(n)
    r = np.concatenate((i, i[1:], i[:-1]))
    c = np.concatenate((i, i[:-1], i[1:]))
    v = np.concatenate((np.full(n, 2.5), np.full(2 * n - 2, -1.0)))
    o = np.lexsort((c, r))
    rp = np.concatenate(([0], np.cumsum(np.bincount(r, minlength=n)))).astype(np.int32)
    return P.CSR(n, rp, c[o].astype(np.int32), v[o])


CASES = {
    "chain": lambda: chain(60000),
    "poisson3d": lambda: P.poisson3d(50),
    "long rows": lambda: P.random_symmetric_pattern(6000, 0.012, 11, weights=(1, 2, 3, 5)),
}


@pytest.mark.parametrize("alternate", [0, 1])
@pytest.mark.parametrize("name", list(CASES))
def test_given_up_and_repeated(name, alternate, monkeypatch):
    """No time at all for the first attempt: waves that have not finished by their first look at the clock (1024
    sweeps) leave, the others and the tiles not yet started follow."""
    print("case", name, alternate, flush=True)
    a = CASES[name]()
    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    monkeypatch.setenv("HEMAMG_HEM_LIMIT", "0")
    monkeypatch.setenv("HEMAMG_HEM_TILE", "64")
    if name == "chain":  # surely longer than that
        monkeypatch.setenv("HEMAMG_TILE_STRICT", "1")
        with pytest.raises(hemamg.AmgError, match="did not finish in time"):
            hemamg.Hierarchy(A, alternate=alternate)
        monkeypatch.delenv("HEMAMG_TILE_STRICT")
    with hemamg.Hierarchy(A, alternate=alternate) as g:
        assert_same_hierarchy(g, oracle.Hierarchy(a, alternate=alternate))


def test_given_up_in_a_batch(monkeypatch):
    systems = [chain(9000), P.poisson3d(17, 13, 11), chain(30011)]
    devs = [hemamg.DeviceCSR.from_host(a, device="cuda:0") for a in systems]
    import torch

    rhs = torch.from_numpy(np.concatenate([P.rhs_uniform(a.n, k) for k, a in enumerate(systems)])).to("cuda:0")
    out = []
    for limit in ("-1", "0"):
        monkeypatch.setenv("HEMAMG_HEM_LIMIT", limit)
        bt = hemamg.Batch.setup(devs, hemamg.amg_params_default())
        try:
            assert bt.status == [hemamg.AMG_OK] * len(systems)
            x, info = bt.solve(rhs, rtol=1e-8, maxit=500)
            out.append(x.cpu().numpy())
        finally:
            bt.close()
    np.testing.assert_array_equal(out[0].view(np.int64), out[1].view(np.int64))


def test_a_long_chain_is_within_the_limit(monkeypatch):
    """A million rows in one chain: 500,000 decisions in the first pass, each waiting for the one before."""
    monkeypatch.setenv("HEMAMG_TILE_STRICT", "1")
    a = chain(1000003)
    A = hemamg.DeviceCSR.from_host(a, device="cuda:0")
    with hemamg.Hierarchy(A) as g:
        s = g.stats()
        print("passes", s["pass_n"], s["match_ms"], flush=True)
        assert_same_hierarchy(g, oracle.Hierarchy(a))
