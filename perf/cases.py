"""Performance cases: what a user of the library has it do, over the range of
sizes, operators and options it is used with.

A case is a dict of plain values:

* ``do``: "solve" (a hierarchy is at hand, one right-hand side), "setup" (a new
  operator: hierarchy and first solve, as the serving loop does on a cache
  miss), "batch" (k right-hand sides against one hierarchy), "vcycle" (one
  application of the preconditioner, for a Krylov method of the user's own);
* ``op``: "poisson" (7-point Laplacian on N^3), "aniso" (constant coefficients
  eps_x, eps_y, 1), "blocks" (coefficients constant on 16^3 blocks), "graph"
  (a random symmetric diagonally dominant matrix of N rows);
* ``precision``: of the hierarchy, "fp64" or "fp32" (CG is always FP64);
* ``scheme``: "v" (V-cycle, 1 + 1 sweeps, Cholesky coarsest solve: the
  default), "k" (K-cycle in flexible CG), "sa" (smoothed aggregation with 4 + 4
  sweeps and the CG coarsest solve: the preconditioner of the paper's GPU runs).

Solves stop at ``rtol``. The right-hand side is uniform in (-1, 1), or, with
``rhs`` = "image", A u for a uniform u.
"""

import math

import numpy as np
import torch

from paper_2006_16147_amd import amg, inputs

DEVICE = "cuda:0"


def _case(do, op, N, precision="fp32", scheme="v", rtol=1e-8, rhs="uniform", **more):
    return {"do": do, "op": op, "N": N, "precision": precision, "scheme": scheme, "rtol": rtol,
            "rhs": rhs, **more}


def listed():
    return [
        # a small system inside a program of its own: launches and latency
        dict(_case("solve", "poisson", 20, "fp64", rtol=1e-6), name="solve_20"),
        # the serving loop's cache hit at a middle size
        dict(_case("solve", "aniso", 96, eps_x=0.05, eps_y=0.4), name="solve_96_aniso"),
        # the benchmark's default workload
        dict(_case("solve", "poisson", 160, "fp64", rhs="image"), name="solve_160"),
        # the largest configuration: 16.7 M rows, varying coefficients
        dict(_case("solve", "blocks", 256, "fp64", rhs="image"), name="solve_blocks_256"),
        # the preconditioner alone
        dict(_case("vcycle", "poisson", 80, "fp64"), name="vcycle_80"),
        # the serving loop's cache misses: the smallest, an odd size, the largest
        dict(_case("setup", "poisson", 32), name="setup_32"),
        dict(_case("setup", "aniso", 101, eps_x=0.3, eps_y=0.01), name="setup_101_aniso"),
        dict(_case("setup", "poisson", 192), name="setup_192"),
        # an irregular matrix: no grid, rows of unequal length
        dict(_case("setup", "graph", 100003, "fp64", rhs="image", degree=9.0), name="setup_graph"),
        # the paper's GPU preconditioner at its 512 k unknowns, stop at 1e-6
        dict(_case("setup", "poisson", 80, "fp64", "sa", rtol=1e-6), name="setup_80_smoothed"),
        # the paper's K-cycle at 512 k unknowns
        dict(_case("solve", "poisson", 80, "fp64", "k", rtol=1e-6), name="solve_80_kcycle"),
        # many right-hand sides
        dict(_case("batch", "poisson", 128, k=32), name="batch_128_k32"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    do = rng.choice(["solve", "solve", "solve", "setup", "setup", "setup", "batch", "vcycle"])
    op = rng.choice(["poisson", "poisson", "aniso", "aniso", "blocks", "graph"])
    precision = rng.choice(["fp64", "fp32"])
    scheme, more, rtol = "v", {}, rng.choice([1e-6, 1e-8])
    if do in ("solve", "setup") and op == "poisson":
        scheme = rng.choice(["v", "v", "k", "sa"])
    hi = {"k": 160, "sa": 96}.get(scheme, 192)
    if do == "batch":
        more["k"] = _log_int(rng, 2, 32)
        hi = 128
    N = _log_int(rng, 12, hi)
    if op == "aniso":
        more["eps_x"] = 10.0 ** rng.uniform(-3.0, 0.0)
        more["eps_y"] = 10.0 ** rng.uniform(-3.0, 0.0)
    elif op == "blocks":
        N = 16 * max(2, round(N / 16))
    elif op == "graph":
        N = _log_int(rng, 1000, 30000 if do == "batch" else 200000)
        more["degree"] = round(rng.uniform(4.0, 14.0), 2)
    rhs = "image" if op in ("blocks", "graph") else rng.choice(["uniform", "image"])
    return _case(do, op, N, precision, scheme, rtol, rhs, **more)


# ---- inputs ----------------------------------------------------------------

def _rows(case):
    return case["N"] if case["op"] == "graph" else case["N"] ** 3


def _operator(case, seed):
    """(row_ptr, col, val) on the GPU. Only "blocks" and "graph" depend on the seed."""
    N = case["N"]
    if case["op"] in ("poisson", "aniso"):
        return inputs.constant_diffusion7_arrays(N, case.get("eps_x", 1.0),
                                                 case.get("eps_y", 1.0), 1.0, torch, DEVICE)
    if case["op"] == "blocks":
        ex, ey = inputs.block_log_uniform_eps(N, 16, np.random.default_rng(seed))
        return inputs.diffusion7_torch(N, ex, ey, 1.0, DEVICE)
    A = inputs.random_spd_graph(N, case["degree"], seed)
    return tuple(torch.from_numpy(a).to(DEVICE) for a in (A.row_ptr, A.col, A.val))


def _uniform(case, seed):
    shape = (_rows(case), case["k"]) if case["do"] == "batch" else (_rows(case),)
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    return torch.rand(shape, generator=g, device=DEVICE, dtype=torch.float64) * 2 - 1


def _product(A, u):
    """A u, one row's terms summed after the other (the same on every run)."""
    row_ptr, col, val = A
    offsets, n, step = row_ptr.long(), u.shape[0], 1 << 21
    columns = []
    for c in [u] if u.dim() == 1 else list(u.T):
        terms = val * c[col]
        columns.append(torch.cat([torch.segment_reduce(terms, "sum", unsafe=True,
                                                       offsets=offsets[r:min(r + step, n) + 1])
                                  for r in range(0, n, step)]))
    return columns[0] if u.dim() == 1 else torch.stack(columns, 1).contiguous()


def _rhs(case, seed, A):
    u = _uniform(case, seed)
    return _product(A, u) if case["rhs"] == "image" else u


def _params(case):
    p = {"precision": amg.FP32 if case["precision"] == "fp32" else amg.FP64}
    if case["scheme"] == "k":
        p["cycle"] = amg.CYCLE_K
    elif case["scheme"] == "sa":
        p.update(smooth_p=1, pre=4, post=4, coarse_solver=amg.COARSE_PCG)
    return p


def prepare(case, seed):
    A = _operator(case, seed)
    s = {"case": case, "A": A, "b": _rhs(case, seed, A), "params": _params(case)}
    if case["do"] != "setup":
        s["h"] = amg.amg_setup(*A, **s["params"])
    return s


# ---- one pass --------------------------------------------------------------

def run(state):
    case, b = state["case"], state["b"]
    if case["do"] == "vcycle":
        z = torch.empty_like(b)
        amg.amg_vcycle_apply(state["h"], b, z)
        return {"z": z}
    x = torch.zeros_like(b)
    if case["do"] == "batch":
        _, infos = amg.amg_pcg_solve_batch(state["h"], b, x, rtol=case["rtol"])
        return {"x": x, "iterations": [i["iterations"] for i in infos]}
    if case["do"] == "solve":
        _, info = amg.amg_pcg_solve(state["h"], b, x, rtol=case["rtol"])
        return {"x": x, "iterations": info["iterations"]}
    h = amg.amg_setup(*state["A"], **state["params"])
    _, info = amg.amg_pcg_solve(h, b, x, rtol=case["rtol"])
    sizes = h.sizes()
    h.close()
    return {"x": x, "iterations": info["iterations"], "sizes": sizes}


# ---- what a pass cannot do without -----------------------------------------

def _iterations(case):
    """About the iterations the stop test takes (as counted on these operators)."""
    n, to6 = _rows(case), case["rtol"] >= 1e-6
    if case["op"] == "graph":
        return 10 if to6 else 14
    if case["scheme"] == "sa":
        return 7 if to6 else 9
    if case["scheme"] == "k":
        return 13 if to6 else 18
    base = {"poisson": 9.0, "aniso": 12.0, "blocks": 15.0}[case["op"]] * n ** 0.1
    return round(base * (0.7 if to6 else 1.0))


def work(case):
    """Every stored matrix entry once per product with it (an iteration: CG, the
    way down and the way up), every vector once per kernel that must follow a
    reduction or another product; a setup reads A and writes each level's
    matrices once."""
    n = _rows(case)
    nnz = n * (case["degree"] + 1) if case["op"] == "graph" else 7 * n - 6 * case["N"] ** 2
    v = 4 if case["precision"] == "fp32" else 8
    opc, sweeps = (2.1, 8) if case["scheme"] == "sa" else (1.143, 2)
    k = case.get("k", 1)
    cycle_bytes = sweeps * opc * (nnz * (v + 4) + 3 * n * v * k)
    cycle_flops = 2 * sweeps * opc * nnz * k
    if case["scheme"] == "k":  # level l is visited 2^(l - 1) times, with two products more
        cycle_bytes *= 1.5
        cycle_flops *= 1.5
    if case["do"] == "vcycle":
        return {"bytes": cycle_bytes + 16 * n, "flops": cycle_flops}
    it = _iterations(case)
    total = {"bytes": it * (cycle_bytes + nnz * 12 + 11 * 8 * n * k),
             "flops": it * (cycle_flops + 2 * nnz * k + 10 * n * k)}
    if case["do"] == "setup":
        total["bytes"] += nnz * 12 + opc * nnz * (12 + 2 * (v + 4)) + 8 * 8 * n
        total["flops"] += 20 * opc * nnz
    return total


# ---- reference values ------------------------------------------------------

def _sine_solve(case, b):
    """Exact solution of the constant-coefficient operators: it is diagonal in
    the product of sine bases."""
    N, k = case["N"], b.shape[1] if b.dim() == 2 else 1
    t = torch.arange(1, N + 1, dtype=torch.float64, device=b.device)
    S = torch.sin(torch.outer(t, t) * (math.pi / (N + 1))) * math.sqrt(2.0 / (N + 1))
    lam = 2.0 - 2.0 * torch.cos(t * (math.pi / (N + 1)))
    ex, ey = case.get("eps_x", 1.0), case.get("eps_y", 1.0)
    d = (lam.view(N, 1, 1) + ey * lam.view(1, N, 1) + ex * lam.view(1, 1, N)).reshape(N ** 3, 1)

    def transform(v):  # S along z, y and x (the grid order is z, y, x)
        v = (S @ v.reshape(N, N * N * k)).reshape(N, N, N * k)
        v = (S @ v.transpose(0, 1).reshape(N, N * N * k)).reshape(N, N, N * k).transpose(0, 1)
        v = v.reshape(N * N, N, k).transpose(0, 1).reshape(N, N * N * k)
        v = (S @ v).reshape(N, N * N, k).transpose(0, 1)
        return v.reshape(N ** 3, k)

    return transform(transform(b.reshape(N ** 3, k)) / d).reshape(b.shape)


def _laplacian(v):
    """The 7-point Laplacian of an N^3 array, zero outside."""
    y = 6.0 * v
    for a in range(3):
        n = v.shape[a]
        y.narrow(a, 1, n - 1).sub_(v.narrow(a, 0, n - 1))
        y.narrow(a, 0, n - 1).sub_(v.narrow(a, 1, n - 1))
    return y


def _cube_vcycle(r, level):
    """The V-cycle where every level's aggregates are the 2 x 2 x 2 cubes: the
    level's matrix is the Laplacian / 2^level, P has entries 8^-1/2."""
    N = r.shape[0]
    scale = 0.5 ** level
    if N ** 3 <= 200:
        flat = {"N": N}
        return _sine_solve(flat, r.reshape(-1)).reshape(N, N, N) / scale
    ones = torch.ones_like(r)
    neighbours = 6.0 * ones - _laplacian(ones)  # number of stored off-diagonals
    m = scale * (6.0 + neighbours)
    z = r / m
    t = r - scale * _laplacian(z)
    h = N // 2
    rc = t.reshape(h, 2, h, 2, h, 2).sum((1, 3, 5)) / math.sqrt(8.0)
    zc = _cube_vcycle(rc, level + 1) / math.sqrt(8.0)
    z = z + zc.reshape(h, 1, h, 1, h, 1).expand(h, 2, h, 2, h, 2).reshape(N, N, N)
    return z + (r - scale * _laplacian(z)) / m


def _halves(N):
    while N ** 3 > 200:
        if N % 2:
            return False
        N //= 2
    return True


def exact(case, seed):
    if case["do"] == "vcycle":
        if case["op"] != "poisson" or not _halves(case["N"]):
            return None
        N = case["N"]
        r = _rhs(case, seed, _operator(case, seed) if case["rhs"] == "image" else None)
        return {"z": _cube_vcycle(r.reshape(N, N, N), 0).reshape(-1)}
    u = _uniform(case, seed)
    x = u if case["rhs"] == "image" else _sine_solve(case, u)
    return {"x": x, "iterations": None, "sizes": None} if case["do"] == "setup" else {
        "x": x, "iterations": None}
