"""Performance cases: the calls a program that uses this library makes, each
through its public entry points, over the sizes and options they come in.

A case is a dict of plain values: `call` names what one pass does,

  step    one system solved once: setup, Krylov solve, destroy
  solve   a Krylov solve on a handle that is kept (new right-hand sides)
  vcycle  one application of a kept preconditioner, z = M^{-1} r
  setup   a preconditioner built and applied once
  batch   many small systems set up and solved together
  serve   requests sent to a running server and waited for

`op` and `nx, ny, nz` say which operator (natural order, x fastest), `fp32`
whether the preconditioner runs in single precision.
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_2007_00056_amd import hemamg

DEV = "cuda"


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # the smallest whole solve, a 2-D Poisson system: launches, host waits and read-backs
        dict(name="step_poisson2d_64", call="step", op="poisson", nx=64, ny=64, nz=1, fp32=False, method="pcg",
             rtol=1e-8),
        # the benchmark's default: a large regular system, all in double
        dict(name="step_poisson3d_128", call="step", op="poisson", nx=128, ny=128, nz=128, fp32=False, method="pcg",
             rtol=1e-10),
        # the largest: smooth, strongly varying coefficients, where matching chains are long
        dict(name="step_vardiff3d_160", call="step", op="vardiff", nx=160, ny=160, nz=160, fp32=True, method="pcg",
             rtol=1e-8),
        # a nonsymmetric system
        dict(name="step_convdiff3d_96", call="step", op="convdiff", nx=96, ny=96, nz=96, fp32=True,
             method="bicgstab", rtol=1e-8),
        # time stepping: one matrix with rough coefficients, a new right-hand side a step; ragged sides
        dict(name="solve_lognormal_61x67x53", call="solve", op="lognormal", nx=61, ny=67, nz=53, fp32=False,
             method="pcg", rtol=1e-8),
        # the same for a nonsymmetric matrix, in double
        dict(name="solve_convdiff_77x45x31", call="solve", op="convdiff", nx=77, ny=45, nz=31, fp32=False,
             method="bicgstab", rtol=1e-8),
        # the preconditioner inside a caller's own Krylov method: large, in double
        dict(name="vcycle_poisson3d_128", call="vcycle", op="poisson", nx=128, ny=128, nz=128, fp32=False),
        # ... an odd size in single precision, coarse levels of irregular shape
        dict(name="vcycle_vardiff_97x101x89", call="vcycle", op="vardiff", nx=97, ny=101, nz=89, fp32=True),
        # ... and small, where every level is bound by latency
        dict(name="vcycle_lognormal_24", call="vcycle", op="lognormal", nx=24, ny=24, nz=24, fp32=True),
        # a preconditioner for a matrix that changes at each step (nonlinear problems): setup and one use
        dict(name="setup_lognormal_91x75x64", call="setup", op="lognormal", nx=91, ny=75, nz=64, fp32=False),
        # many small systems at once, sides 16 to 32
        dict(name="batch_32_sides_16_32", call="batch", op="lognormal", count=32, side_min=16, side_max=32, fp32=True,
             method="pcg", rtol=1e-8),
        # served requests, the stream's sides up to 64
        dict(name="serve_64_sides_16_64", call="serve", op="lognormal", count=64, side_min=16, side_max=64, fp32=True,
             method="pcg", rtol=1e-8),
    ]


def draw(rng):
    """One more case: rows log-uniform over the listed range, sides unequal and odd as they fall."""
    call = rng.choice(["step", "step", "solve", "solve", "vcycle", "vcycle", "setup", "batch", "serve"])
    fp32 = rng.random() < 0.5
    if call in ("batch", "serve"):
        lo = rng.randint(12, 20)
        return dict(call=call, op="lognormal", count=rng.randint(8, 32 if call == "batch" else 64), side_min=lo,
                    side_max=lo + rng.randint(6, 24 if call == "batch" else 40), fp32=fp32, method="pcg", rtol=1e-8)
    flat = rng.random() < 0.2
    op = "poisson" if flat else rng.choice(["poisson", "vardiff", "lognormal", "convdiff"])
    rows = math.exp(rng.uniform(math.log(4000), math.log(2.0e6)))
    if flat:
        a = rng.uniform(-0.4, 0.4)
        nx, ny, nz = round(math.sqrt(rows) * math.exp(a)), round(math.sqrt(rows) * math.exp(-a)), 1
    else:
        a, b, side = rng.uniform(-0.3, 0.3), rng.uniform(-0.3, 0.3), rows ** (1 / 3)
        nx, ny, nz = round(side * math.exp(a)), round(side * math.exp(b)), round(side * math.exp(-a - b))
    c = dict(call=call, op=op, nx=nx, ny=ny, nz=nz, fp32=fp32)
    if call in ("step", "solve"):
        c.update(method="bicgstab" if op == "convdiff" else "pcg", rtol=rng.choice([1e-8, 1e-10]))
    return c


# ---------------------------------------------------------------- operators

def grid_csr(diag, west, east, south, north, down, up, shape):
    """CSR of a 5- or 7-point operator on the interior of a box; boundary
    neighbours drop out.  Coefficients: numbers or (nz, ny, nx) tensors."""
    nz, ny, nx = shape
    n = nx * ny * nz
    idx = torch.arange(n, device=DEV)
    x, y, z = idx % nx, (idx // nx) % ny, idx // (nx * ny)
    parts = [(south, -nx, y > 0), (west, -1, x > 0), (diag, 0, x >= 0), (east, 1, x < nx - 1),
             (north, nx, y < ny - 1)]
    if nz > 1:
        parts = [(down, -nx * ny, z > 0)] + parts + [(up, nx * ny, z < nz - 1)]
    keep = torch.stack([m for _, _, m in parts], 1)
    cols = torch.stack([idx + d for _, d, _ in parts], 1)[keep].to(torch.int32)
    full = torch.ones(n, dtype=torch.float64, device=DEV)
    vals = torch.stack([(c.reshape(-1) if torch.is_tensor(c) else c * full) for c, _, _ in parts], 1)[keep]
    rp = torch.zeros(n + 1, dtype=torch.int32, device=DEV)
    rp[1:] = keep.sum(1).cumsum(0)
    return rp, cols, vals


def fv_csr(tx, ty, tz, shape):
    """Finite-volume diffusion from face values (the first and last face of a
    line are the Dirichlet walls)."""
    diag = tx[:, :, :-1] + tx[:, :, 1:] + ty[:, :-1] + ty[:, 1:] + tz[:-1] + tz[1:]
    return grid_csr(diag, -tx[:, :, :-1], -tx[:, :, 1:], -ty[:, :-1], -ty[:, 1:], -tz[:-1], -tz[1:], shape)


def operator(op, nx, ny, nz, gen):
    shape = (nz, ny, nx)
    if op == "poisson":
        return grid_csr(6.0 if nz > 1 else 4.0, -1.0, -1.0, -1.0, -1.0, -1.0, -1.0, shape)
    if op == "convdiff":  # first-order upwind, velocity (1, 1/2, 1/4), cell Peclet number 10
        return grid_csr(23.5, -11.0, -1.0, -6.0, -1.0, -3.5, -1.0, shape)
    faces = [(nz, ny, nx + 1), (nz, ny + 1, nx), (nz + 1, ny, nx)]
    if op == "lognormal":  # independent face values exp(N(0, 1)), walls at half a cell
        t = [torch.exp(torch.randn(f, generator=gen, device=DEV, dtype=torch.float64)) for f in faces]
        for d, f in zip((2, 1, 0), t):
            f.select(d, 0).mul_(2.0)
            f.select(d, -1).mul_(2.0)
        return fv_csr(*t, shape)
    if op != "vardiff":
        raise ValueError(op)
    # coefficient exp(g): g a smooth Gaussian field, standard deviation 1.5, correlation length 8 cells
    g = torch.fft.fftn(torch.randn(shape, generator=gen, device=DEV, dtype=torch.float64))
    for d, m in enumerate(shape):
        k = 2.0 * math.pi * torch.fft.fftfreq(m, device=DEV, dtype=torch.float64)
        f = torch.exp(-0.5 * (8.0 / math.sqrt(2.0)) ** 2 * k * k)
        g = g * f.reshape([-1 if e == d else 1 for e in range(3)])
    g = torch.fft.ifftn(g).real
    g = g - g.mean()
    g = g * (1.5 / g.std())
    t = []
    for d, f in zip((2, 1, 0), faces):
        m = shape[d]
        face = torch.empty(f, device=DEV, dtype=torch.float64)
        face.narrow(d, 1, m - 1).copy_(torch.exp(0.5 * (g.narrow(d, 0, m - 1) + g.narrow(d, 1, m - 1))))
        face.select(d, 0).copy_(2.0 * torch.exp(g.select(d, 0)))
        face.select(d, -1).copy_(2.0 * torch.exp(g.select(d, -1)))
        t.append(face)
    return fv_csr(*t, shape)


def sides(case):
    """Sides of a batch's or stream's systems: log-uniform over the case's range, the same for every seed."""
    r = np.random.default_rng(case["count"])
    u = r.uniform(math.log(case["side_min"]), math.log(case["side_max"]), case["count"])
    return [int(s) for s in np.rint(np.exp(u))]


def inputs(case, seed):
    """The systems (CSR triples) and right-hand sides uniform on [-1, 1], one after another."""
    gen = torch.Generator(device=DEV).manual_seed(seed)
    if "count" in case:
        systems = [operator(case["op"], s, s, s, gen) for s in sides(case)]
    else:
        systems = [operator(case["op"], case["nx"], case["ny"], case["nz"], gen)]
    n = sum(rp.numel() - 1 for rp, _, _ in systems)
    return systems, 2.0 * torch.rand(n, generator=gen, device=DEV, dtype=torch.float64) - 1.0


# ---------------------------------------------------------------- what runs

class Server:
    def __init__(self, fp32):
        cfg = hemamg.amg_server_config_default(workers=8, batch=32)
        cfg.params.precond_fp32 = int(fp32)
        self.h = hemamg.amg_server_create(cfg)

    def __del__(self):
        hemamg.amg_server_destroy(self.h)


def prepare(case, seed):
    systems, b = inputs(case, seed)
    s = dict(case=case, b=b, A=[hemamg.DeviceCSR(*a) for a in systems])
    fp32 = int(case["fp32"])
    if case["call"] in ("solve", "vcycle"):
        s["h"] = hemamg.Hierarchy(s["A"][0], precond_fp32=fp32)
    elif case["call"] == "serve":
        s["server"] = Server(fp32)
    return s


def run(s):
    case, b, A = s["case"], s["b"], s["A"]
    call, fp32 = case["call"], int(case["fp32"])
    if call == "step":
        with hemamg.Hierarchy(A[0], precond_fp32=fp32) as h:
            return h.solve(b, method=case["method"], rtol=case["rtol"])[0]
    if call == "solve":
        return s["h"].solve(b, method=case["method"], rtol=case["rtol"])[0]
    if call == "vcycle":
        return s["h"].vcycle(b)
    if call == "setup":
        with hemamg.Hierarchy(A[0], precond_fp32=fp32) as h:
            return {"z": h.vcycle(b), "rows": [hemamg.amg_level_size(h.h, k)[0] for k in range(h.nlevels)]}
    if call == "batch":
        with hemamg.Batch.setup(A, precond_fp32=fp32) as bt:
            x, info = bt.solve(b, method=case["method"], rtol=case["rtol"])
        return {"x": x, "status": [i["status"] for i in info]}
    x = torch.zeros_like(b)
    srv, o, tickets = s["server"].h, 0, []
    for a in A:
        tickets.append(hemamg.amg_server_submit(srv, a, b[o:o + a.n], x[o:o + a.n], hemamg.PCG, case["rtol"], 1000))
        o += a.n
    info = [hemamg.amg_server_wait(srv, t) for t in tickets]
    return {"x": x, "failed": sum(i["status"] != hemamg.AMG_OK for i in info)}


# ---------------------------------------------------------------- what a pass cannot do without

# PCG (BiCGStab for convdiff) iterations per digit of the tolerance and square root of the side, from runs
ITERATIONS = dict(poisson=0.45, vardiff=1.0, lognormal=0.6, convdiff=0.24)


def work(case):
    """One pass: a V-cycle reads level 0 twice (residual after the
    presmoothing, postsmoothing) and, with aggregates of up to four rows, a
    third as much again on the coarse levels; a PCG iteration adds one more
    product and its vectors, a BiCGStab iteration is two of each.  A setup
    reads the matrix and writes coarse operators of a third of its size."""
    dims = [(s, s, s) for s in sides(case)] if "count" in case else [(case["nx"], case["ny"], case["nz"])]
    e = 4 if case["fp32"] else 8
    nbytes = flops = 0.0
    for nx, ny, nz in dims:
        n = nx * ny * nz
        nnz = n + 2 * (3 * n - ny * nz - nx * nz - nx * ny) if nz > 1 else n + 2 * (2 * n - ny - nx)
        read = 12.0 * nnz + 4.0 * n
        cycle = (4.0 / 3.0) * 2.0 * ((e + 4.0) * nnz + 4.0 * n) + 16.0 * n
        cycle_flops = (4.0 / 3.0) * 2.0 * (2.0 * nnz + 3.0 * n)
        if case["call"] in ("step", "setup", "batch", "serve"):
            nbytes += (4.0 / 3.0) * read
            flops += (8.0 / 3.0) * nnz
        if case["call"] in ("vcycle", "setup"):
            nbytes += cycle
            flops += cycle_flops
        else:
            side = n ** (1 / 3) if nz > 1 else math.sqrt(n)
            its = ITERATIONS[case["op"]] * -math.log10(case["rtol"]) * math.sqrt(side)
            its *= 2.0 if case["method"] == "bicgstab" else 1.0
            nbytes += its * (cycle + read + 80.0 * n)
            flops += its * (cycle_flops + 2.0 * nnz + 12.0 * n)
    return {"bytes": nbytes, "flops": flops}


# ---------------------------------------------------------------- the same in 64 bits, without the library

def matvec(rp, ci, v):
    rows = torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), torch.diff(rp.long()))
    A = torch.sparse_csr_tensor(rp.long(), ci.long(), v)
    d = torch.zeros(rp.numel() - 1, dtype=torch.float64, device=DEV)
    on = ci.long() == rows
    d[rows[on]] = v[on]
    return (lambda x: (A @ x[:, None])[:, 0]), d


def solve_exact(rp, ci, v, b, symmetric):
    """x = A^{-1} b by Jacobi-preconditioned CG or BiCGStab far below the cases' tolerances."""
    mul, d = matvec(rp, ci, v)
    x, r = torch.zeros_like(b), b.clone()
    goal = 1e-14 * float(b.norm())
    p, rb = (r / d, None) if symmetric else (r.clone(), r.clone())
    rho = r @ (p if symmetric else rb)
    for it in range(20000):
        if it % 25 == 0 and float(r.norm()) <= goal:
            break
        if symmetric:
            q = mul(p)
            a = rho / (p @ q)
            x, r = x + a * p, r - a * q
            z = r / d
            rho, old = r @ z, rho
            p = z + (rho / old) * p
        else:
            ph = p / d
            q = mul(ph)
            a = rho / (rb @ q)
            s = r - a * q
            sh = s / d
            t = mul(sh)
            w = (t @ s) / (t @ t)
            x, r = x + a * ph + w * sh, s - w * t
            rho, old = rb @ r, rho
            p = r + (rho / old) * (a / w) * (p - w * q)
    return x


def match(rp, ci, v):
    """Algorithm 2, row by row: each unmatched row takes its heaviest unmatched
    neighbour, lowest index on ties.  Returns the aggregate of every row."""
    n = rp.numel() - 1
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), torch.diff(rp))
    up = (ci > rows) & (v != 0)  # a lower neighbour is matched, or was left alone for good
    r, c, w = rows[up], ci[up], v[up].abs()
    o = torch.argsort(w, descending=True, stable=True)  # columns ascend within a row
    o = o[torch.argsort(r[o], stable=True)]
    start = torch.searchsorted(r[o], torch.arange(n + 1, device=DEV)).tolist()
    nb = c[o].tolist()
    agg, nc = [-1] * n, 0
    for u in range(n):
        if agg[u] < 0:
            agg[u] = nc
            for k in range(start[u], start[u + 1]):
                if agg[nb[k]] < 0:
                    agg[nb[k]] = nc
                    break
            nc += 1
    return torch.tensor(agg, device=DEV), nc


def coarse(rp, ci, v, agg, nc):
    rows = torch.repeat_interleave(torch.arange(rp.numel() - 1, device=DEV), torch.diff(rp))
    key, at = torch.unique(agg[rows] * nc + agg[ci], return_inverse=True)
    val = torch.zeros(key.numel(), dtype=torch.float64, device=DEV).index_add_(0, at, v)
    crp = torch.searchsorted(key, torch.arange(nc + 1, device=DEV) * nc)
    return crp, key % nc, val


def vcycle_exact(rp, ci, v, r):
    """z = M^{-1} r and the rows of every level (two matching passes a level, weight 2/3, one sweep each way)."""
    lev, A = [], (rp.long(), ci.long(), v)
    while A[0].numel() - 1 > 64:
        n = A[0].numel() - 1
        a1, n1 = match(*A)
        B = coarse(*A, a1, n1)
        a2, n2 = match(*B)
        if n2 == n or (n2 >= 0.9 * n and n <= 4096):
            break
        lev.append((A, a2[a1]))
        A = coarse(*B, a2, n2)
    m = A[0].numel() - 1
    dense = torch.zeros(m, m, dtype=torch.float64, device=DEV)
    dense[torch.repeat_interleave(torch.arange(m, device=DEV), torch.diff(A[0])), A[1]] = A[2]

    def cycle(k, f):
        if k == len(lev):
            return torch.linalg.solve(dense, f)
        (mul, d), agg = matvec(*lev[k][0]), lev[k][1]
        x = (2.0 / 3.0) * f / d
        nc = lev[k + 1][0][0].numel() - 1 if k + 1 < len(lev) else m
        fc = torch.zeros(nc, dtype=torch.float64, device=DEV).index_add_(0, agg, f - mul(x))
        x = x + cycle(k + 1, fc)[agg]
        return x + (2.0 / 3.0) * (f - mul(x)) / d

    return cycle(0, r), [a[0].numel() - 1 for a, _ in lev] + [m]


def exact(case, seed):
    systems, b = inputs(case, seed)
    if case["call"] in ("vcycle", "setup"):
        z, rows = vcycle_exact(*systems[0], b)
        return z if case["call"] == "vcycle" else {"z": z, "rows": rows}
    if "count" in case:  # the systems side by side as one block-diagonal matrix
        n = np.cumsum([0] + [rp.numel() - 1 for rp, _, _ in systems]).tolist()
        e = np.cumsum([0] + [ci.numel() for _, ci, _ in systems]).tolist()
        rp = torch.cat([a[0][:-1].long() + o for a, o in zip(systems, e)] + [torch.tensor([e[-1]], device=DEV)])
        ci = torch.cat([a[1].long() + o for a, o in zip(systems, n)])
        x = solve_exact(rp, ci, torch.cat([a[2] for a in systems]), b, True)
        return {"x": x, "status" if case["call"] == "batch" else "failed": None}
    return solve_exact(*systems[0], b, case["op"] != "convdiff")
