"""The work that a user has this library do, as cases that can be timed.

A case is a dict of plain values.  "kind" says which public entry points a
pass goes through, "matrix" with its sizes says on which operator:

  solve    Hierarchy.solve on a hierarchy that the program keeps: one
           right-hand side after another against the same matrix
  step     Hierarchy + solve + close: one step of a program whose matrix
           changes from step to step (the benchmark's step)
  precond  Hierarchy.precond: one cycle, inside a program's own Krylov loop
  grad     the differentiable solve: forward, and backward to the gradients of
           the matrix values and of the right-hand side
  match    one matching sweep: the mates and the edge weights

  poisson2d, poisson3d   5- and 7-point Laplacians, Dirichlet
  diffusion3d            cell-centred finite volumes, log-normal coefficients
                         (sigma = std of ln kappa), harmonic faces, z faces
                         scaled by z_scale
  elasticity3d           Q1 hexahedra, nx^3 elements, x = 0 face clamped, 20%
                         of the elements nearly incompressible
  graph                  a random weighted graph Laplacian plus a positive
                         diagonal: rows of irregular length and no order

Matrices and vectors are made on the GPU from the seed alone.
"""
import itertools
import math
import time

import numpy as np
import torch

from paper_1810_04221_amd import bcm

DEV = "cuda"


# ---------------------------------------------------------------- the cases
def _case(name, kind, matrix, nx, ny=0, nz=0, sigma=0.0, z_scale=1.0, precision="fp64", cycle="V", tol=1e-10,
          max_coarse=0, min_ratio=0.0):
    return dict(name=name, kind=kind, matrix=matrix, nx=nx, ny=ny or nx, nz=nz or (1 if matrix == "poisson2d" else nx),
                sigma=sigma, z_scale=z_scale, precision=precision, cycle=cycle, tol=tol, max_coarse=max_coarse,
                min_ratio=min_ratio)


def listed():
    return [
        # the smallest calls: a few thousand unknowns, where launches and latency count
        _case("solve poisson2d 64x64", "solve", "poisson2d", 64),
        _case("step poisson2d 97x61 f32", "step", "poisson2d", 97, 61, precision="fp32"),
        # the benchmark's workload: setup + solve, a million unknowns, float32 cycle
        _case("step poisson3d 100 f32", "step", "poisson3d", 100, precision="fp32", max_coarse=99),
        # ordinary sizes, ragged in every direction, under the W-cycle
        _case("solve poisson3d 63x50x77 W", "solve", "poisson3d", 63, 50, 77, cycle="W"),
        # the preconditioner inside a program's own Krylov loop
        _case("precond poisson3d 100", "precond", "poisson3d", 100, max_coarse=99),
        # variable coefficients under the default stopping rule, a new matrix per step
        _case("step diffusion3d 64 f32", "step", "diffusion3d", 64, sigma=1.0, precision="fp32"),
        # the same, two million unknowns, one matrix and many right-hand sides
        _case("solve diffusion3d 128 f32", "solve", "diffusion3d", 128, sigma=1.0, precision="fp32"),
        # the largest: strongly heterogeneous and anisotropic, four million unknowns
        _case("step diffusion3d 160 aniso", "step", "diffusion3d", 160, sigma=2.0, z_scale=1e-2),
        # rows of about 80 entries: elasticity
        _case("step elasticity3d 32 f32", "step", "elasticity3d", 32, precision="fp32"),
        # no grid at all: irregular rows, no locality
        _case("step graph 50000", "step", "graph", 50000),
        # forward and backward of the differentiable solve, odd sizes, the ratio rule
        _case("grad diffusion3d 77x59x83 f32", "grad", "diffusion3d", 77, 59, 83, sigma=1.0, precision="fp32",
              min_ratio=2.0),
        # a matching sweep alone, a million vertices
        _case("match diffusion3d 101x99x103", "match", "diffusion3d", 101, 99, 103, sigma=1.0),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["solve", "solve", "step", "step", "precond", "grad", "match"])
    matrix = rng.choice(["poisson2d", "poisson3d", "diffusion3d", "diffusion3d", "elasticity3d", "graph"])
    # one pattern and other values from seed to seed, where the values come back
    if (kind == "match" and matrix.startswith("poisson")) or (kind in ("match", "grad") and matrix == "graph"):
        matrix = "diffusion3d"
    precision = "fp64" if kind in ("precond", "match") else rng.choice(["fp64", "fp32"])
    c = dict(kind=kind, matrix=matrix, sigma=0.0, z_scale=1.0, precision=precision, cycle="V", tol=1e-10, max_coarse=0,
             min_ratio=0.0, ny=1, nz=1)
    if matrix == "poisson2d":
        c["nx"], c["ny"] = _log_int(rng, 40, 1000), _log_int(rng, 40, 1000)
    elif matrix == "elasticity3d":
        c["nx"] = c["ny"] = c["nz"] = rng.randint(8, 40)
    elif matrix == "graph":
        c["nx"] = _log_int(rng, 2000, 120000)
    else:
        m = _log_int(rng, 20, 100 if kind == "grad" else 145)  # the mean side; the three differ by up to a fifth
        for k in ("nx", "ny", "nz"):
            c[k] = max(8, int(round(m * rng.uniform(0.9, 1.1))))
    if matrix == "diffusion3d":
        c["sigma"] = rng.choice([1.0, 2.0])
        c["z_scale"] = rng.choice([1.0, 1.0, 1e-2])
        c["min_ratio"] = rng.choice([0.0, 0.0, 2.0])
    elif matrix == "poisson3d" and kind != "match":
        c["cycle"] = rng.choice(["V", "V", "W"])
    return c


# ---------------------------------------------------------------- operators
def _csr(cols, vals, mask):
    """CSR arrays from (rows, slots) arrays whose columns ascend along a row."""
    rp = torch.zeros(mask.shape[0] + 1, dtype=torch.int64, device=DEV)
    rp[1:] = mask.sum(1).cumsum(0)
    return rp.to(torch.int32), cols[mask].to(torch.int32), vals[mask].contiguous()


def _grid(case, seed):
    """5- and 7-point operators on an nx * ny * nz grid, x fastest."""
    nx, ny, nz = case["nx"], case["ny"], case["nz"]
    n = nx * ny * nz
    two_d = case["matrix"] == "poisson2d"
    idx = torch.arange(n, device=DEV).reshape(nz, ny, nx)
    if case["matrix"] == "diffusion3d":
        gen = torch.Generator(device=DEV).manual_seed(seed)
        kap = torch.exp(case["sigma"] * torch.randn(nz, ny, nx, dtype=torch.float64, device=DEV, generator=gen))
    else:
        kap = None
    lo, hi = {}, {}  # transmissibility of each cell's lower and upper face, by axis (0 = none)
    diag = torch.zeros(nz, ny, nx, dtype=torch.float64, device=DEV)
    for axis, scale in ((2, 1.0), (1, 1.0), (0, case["z_scale"])):
        if two_d and axis == 0:
            continue
        m = (nz, ny, nx)[axis]
        full = torch.zeros(nz, ny, nx, dtype=torch.float64, device=DEV)
        if kap is None:
            diag += 2.0
            up, down = full.clone(), full.clone()
            up.narrow(axis, 0, m - 1).fill_(1.0)
            down.narrow(axis, 1, m - 1).fill_(1.0)
        else:
            ka, kb = kap.narrow(axis, 0, m - 1), kap.narrow(axis, 1, m - 1)
            T = 2.0 * ka * kb / (ka + kb) * scale
            up, down = full.clone(), full.clone()
            up.narrow(axis, 0, m - 1).copy_(T)
            down.narrow(axis, 1, m - 1).copy_(T)
            diag += up + down
            diag.narrow(axis, 0, 1).add_(2.0 * kap.narrow(axis, 0, 1) * scale)
            diag.narrow(axis, m - 1, 1).add_(2.0 * kap.narrow(axis, m - 1, 1) * scale)
        lo[axis], hi[axis] = down, up
    off, val, ok = [], [], []
    pos = torch.meshgrid(*(torch.arange(m, device=DEV) for m in (nz, ny, nx)), indexing="ij")
    stride = {2: 1, 1: nx, 0: nx * ny}
    for axis in (0, 1, 2):
        if axis in lo:
            off.append(-stride[axis]), val.append(-lo[axis]), ok.append(pos[axis] > 0)
    off.append(0), val.append(diag), ok.append(torch.ones_like(diag, dtype=torch.bool))
    for axis in (2, 1, 0):
        if axis in hi:
            off.append(stride[axis]), val.append(-hi[axis]), ok.append(pos[axis] < (nz, ny, nx)[axis] - 1)
    cols = idx.reshape(n, 1) + torch.tensor(off, device=DEV)
    return _csr(cols, torch.stack([v.reshape(n) for v in val], 1), torch.stack([o.reshape(n) for o in ok], 1))


def _q1_stiffness(nu, h, E=1.0):
    """24 x 24 stiffness of a cube of side h (2 x 2 x 2 Gauss points), local dof 3 a + component."""
    lam, mu = E * nu / ((1.0 + nu) * (1.0 - 2.0 * nu)), E / (2.0 * (1.0 + nu))
    D = np.zeros((6, 6))
    D[:3, :3] = lam
    D[np.arange(3), np.arange(3)] += 2.0 * mu
    D[3:, 3:] = np.diag([mu] * 3)
    s = np.array([[2.0 * ((a >> k) & 1) - 1.0 for k in range(3)] for a in range(8)])
    K = np.zeros((24, 24))
    for g in itertools.product((-1.0 / math.sqrt(3.0), 1.0 / math.sqrt(3.0)), repeat=3):
        B = np.zeros((6, 24))
        for a in range(8):
            t = 1.0 + s[a] * np.array(g)
            d = s[a] * np.array([t[1] * t[2], t[0] * t[2], t[0] * t[1]]) / 8.0 * (2.0 / h)
            for r, c, v in ((0, 0, d[0]), (1, 1, d[1]), (2, 2, d[2]), (3, 1, d[2]), (3, 2, d[1]), (4, 0, d[2]),
                            (4, 2, d[0]), (5, 0, d[1]), (5, 1, d[0])):
                B[r, 3 * a + c] = v
        K += B.T @ D @ B * (h / 2.0) ** 3
    return 0.5 * (K + K.T)


def _elasticity(case, seed):
    ne = case["nx"]
    N, h = ne + 1, 1.0 / ne
    gen = torch.Generator(device=DEV).manual_seed(seed)
    soft = torch.zeros(ne ** 3, dtype=torch.bool, device=DEV)
    soft[torch.randperm(ne ** 3, device=DEV, generator=gen)[: int(round(0.2 * ne ** 3))]] = True
    Ks = torch.tensor(np.stack([_q1_stiffness(0.3, h), _q1_stiffness(0.45, h)]), device=DEV)
    which = soft.long().reshape(ne, ne, ne)
    # node blocks: blk[z, y, x, neighbour (27), 3, 3], summed element by element in one order
    blk = torch.zeros(N, N, N, 27, 3, 3, dtype=torch.float64, device=DEV)
    for a in range(8):
        ax, ay, az = a & 1, (a >> 1) & 1, (a >> 2) & 1
        for b in range(8):
            dx, dy, dz = (b & 1) - ax, ((b >> 1) & 1) - ay, ((b >> 2) & 1) - az
            k = (dz + 1) * 9 + (dy + 1) * 3 + dx + 1
            # element (z, y, x) has its corner a at node (z + az, y + ay, x + ax)
            view = blk[az:az + ne, ay:ay + ne, ax:ax + ne, k]
            view += Ks[:, 3 * a:3 * a + 3, 3 * b:3 * b + 3][which]
    # free nodes: x > 0, numbered x fastest
    blk = blk[:, :, 1:].reshape(-1, 27, 3, 3)
    nn = blk.shape[0]
    z, y, x = torch.meshgrid(torch.arange(N, device=DEV), torch.arange(N, device=DEV),
                             torch.arange(1, N, device=DEV), indexing="ij")
    z, y, x = z.reshape(-1, 1), y.reshape(-1, 1), x.reshape(-1, 1)
    d = torch.tensor([(i, j, k) for i in (-1, 0, 1) for j in (-1, 0, 1) for k in (-1, 0, 1)], device=DEV)
    zz, yy, xx = z + d[:, 0], y + d[:, 1], x + d[:, 2]
    ok = (zz >= 0) & (zz < N) & (yy >= 0) & (yy < N) & (xx >= 1) & (xx < N)
    nb = (zz * N + yy) * ne + (xx - 1)
    three = torch.arange(3, device=DEV)
    cols = (3 * nb[:, None, :, None] + three).expand(nn, 3, 27, 3).reshape(3 * nn, 81)
    mask = ok[:, None, :, None].expand(nn, 3, 27, 3).reshape(3 * nn, 81)
    return _csr(cols, blk.permute(0, 2, 1, 3).reshape(3 * nn, 81), mask)


def _graph(case, seed):
    n = case["nx"]
    rng = np.random.default_rng(seed)
    lo, hi = rng.integers(0, n, 5 * n), rng.integers(0, n, 5 * n)
    lo, hi = np.concatenate([lo, np.arange(n - 1)]), np.concatenate([hi, np.arange(1, n)])
    keep = lo != hi
    key = np.unique(np.minimum(lo, hi)[keep] * n + np.maximum(lo, hi)[keep])
    lo, hi = key // n, key % n
    v = rng.uniform(0.1, 1.0, len(lo))
    d = np.bincount(lo, v, n) + np.bincount(hi, v, n) + rng.uniform(0.05, 0.5, n)
    r = np.concatenate([lo, hi, np.arange(n)])
    c = np.concatenate([hi, lo, np.arange(n)])
    a = np.concatenate([-v, -v, d])
    order = np.argsort(r * n + c)
    rp = np.concatenate([[0], np.cumsum(np.bincount(r, minlength=n))])
    return (torch.tensor(rp, dtype=torch.int32, device=DEV), torch.tensor(c[order], dtype=torch.int32, device=DEV),
            torch.tensor(a[order], device=DEV))


def _inputs(case, seed):
    make = {"elasticity3d": _elasticity, "graph": _graph}.get(case["matrix"], _grid)
    rp, ci, va = make(case, seed)
    n = rp.numel() - 1
    gen = torch.Generator(device=DEV).manual_seed(seed + 1)
    b = torch.rand(n, dtype=torch.float64, device=DEV, generator=gen) * 2.0 - 1.0
    return rp, ci, va, b


def _target(b):
    """The gradient cases' target: another vector of the same distribution."""
    return b.flip(0).contiguous()


def _options(case):
    return dict(precision=case["precision"], cycle=case["cycle"], max_coarse=case["max_coarse"],
                min_ratio=case["min_ratio"])


# ---------------------------------------------------------------- what is timed
def prepare(case, seed):
    rp, ci, va, b = _inputs(case, seed)
    s = dict(case=case, rp=rp, ci=ci, va=va, b=b)
    if case["kind"] in ("solve", "precond", "grad"):
        s["h"] = bcm.Hierarchy(rp, ci, va, adjoint_tol=case["tol"], **_options(case))
    if case["kind"] == "grad":
        s["va"] = va.clone().requires_grad_(True)
        s["b"] = b.clone().requires_grad_(True)
        s["target"] = _target(b)
    return s


def run(state):
    case, b = state["case"], state["b"]
    kind = case["kind"]
    if kind == "solve":
        return state["h"].solve(b, tol=case["tol"])
    if kind == "step":
        h = bcm.Hierarchy(state["rp"], state["ci"], state["va"], **_options(case))
        x = h.solve(b, tol=case["tol"])
        h.close()
        return x
    if kind == "precond":
        return state["h"].precond(b)
    if kind == "match":
        mate, c = bcm.match(state["rp"], state["ci"], state["va"])
        return {"mate": mate, "weights": c}
    x = bcm.solve(state["va"], b, state["h"], case["tol"])
    loss = 0.5 * (x - state["target"]).square().sum()
    gval, gb = torch.autograd.grad(loss, (state["va"], b))
    return {"x": x.detach(), "dval": gval, "db": gb}


def _size(case):
    if case["matrix"] == "graph":
        return case["nx"], 13.0 * case["nx"]
    if case["matrix"] == "elasticity3d":
        m = case["nx"]
        return 3 * m * (m + 1) ** 2, 9.0 * (3 * m - 2) * (3 * m + 1) ** 2
    n = case["nx"] * case["ny"] * case["nz"]
    return n, (5.0 if case["matrix"] == "poisson2d" else 7.0) * n


def work(case):
    """The matrix and the vectors read once and the results written once; one
    product with the matrix (an iterative solve needs many, as its method has it)."""
    n, z = _size(case)
    read, written, products = 12.0 * z + 4.0 * n + 8.0 * n, 8.0 * n, 1.0
    if case["kind"] == "grad":  # forward and backward, the target; both gradients
        read, written, products = read + 8.0 * n, 16.0 * n + 8.0 * z, 3.0
    elif case["kind"] == "match":  # (no right-hand side) the mates and the weights; six operations a weight
        read, written, products = 12.0 * z + 4.0 * n, 4.0 * n + 8.0 * z, 3.0
    return {"bytes": read + written, "flops": 2.0 * z * products}


# ---------------------------------------------------------------- in 64 bits
def _cg(A, d, b, seconds):
    """A x = b by diagonally preconditioned CG, restarted from the true
    residual until that stops falling; None when it takes too long."""
    end = time.monotonic() + seconds
    x = torch.zeros_like(b)
    best, r = math.inf, b
    bn = float(b.norm())
    while True:
        y = torch.zeros_like(b)
        z = r / d
        p, rz, rr0 = z.clone(), torch.dot(r, z), float(r.norm())
        q = r.clone()
        for it in range(200000):
            Ap = A @ p
            al = rz / torch.dot(p, Ap)
            y += al * p
            q -= al * Ap
            z = q / d
            new = torch.dot(q, z)
            p = z + (new / rz) * p
            rz = new
            if it % 50 == 49:
                if float(q.norm()) <= 1e-9 * rr0:
                    break
                if time.monotonic() > end:
                    return None
        x = x + y
        r = b - A @ x
        now = float(r.norm()) / bn
        if now > 0.5 * best or now < 1e-15:
            return x
        best = now


def exact(case, seed):
    if case["kind"] == "precond":
        return None
    rp, ci, va, b = _inputs(case, seed)
    n = rp.numel() - 1
    rows = torch.repeat_interleave(torch.arange(n, device=DEV), (rp[1:] - rp[:-1]).long())
    diag = torch.empty(n, dtype=torch.float64, device=DEV)
    on = rows == ci
    diag[rows[on]] = va[on]
    if case["kind"] == "match":  # w = 1
        c = 1.0 - 2.0 * va / (diag[torch.minimum(rows, ci.long())] + diag[torch.maximum(rows, ci.long())])
        return {"mate": None, "weights": torch.where(on, torch.zeros_like(c), c)}
    A = torch.sparse_csr_tensor(rp, ci, va, size=(n, n))
    x = _cg(A, diag, b, 9.0 if case["kind"] == "grad" else 12.0)
    if case["kind"] != "grad" or x is None:
        return x
    lam = _cg(A, diag, x - _target(b), 9.0)
    if lam is None:
        return None
    return {"x": x, "dval": -lam[rows] * x[ci.long()], "db": lam}
