"""Timed workloads of the UA-AMG library: setup, solve and preconditioner calls on the
problems that the tests, the benchmark and the serving loop use.

A case names one call pattern (``call``) on one problem:

* ``setup_solve``: a new matrix is set up, solved for one right-hand side and released
  (the benchmark's step, and a first request for a problem in the serving loop);
* ``solve``: one right-hand side (or a batch) on a hierarchy that the program keeps
  (time stepping, a repeated request);
* ``kcycle``: one application of the preconditioner inside a caller's own Krylov method;
* ``setup_kcycle``: a new matrix is set up and its preconditioner applied once;
* ``group``: many small problems solved in one launch.

Problems: 2D and 3D (2d+1)-point grid Laplacians with jittered weights (``gx``, ``gy``,
``gz``; gz = 0 for 2D) and random geometric graphs (``points``).
"""
from __future__ import annotations

import math

import numpy as np
import torch

from paper_1302_2547_amd import amg, inputs

FP32 = amg.AMG_PREC_FP32_INNER
MAX_LEVELS = 40  # the library's default limit


def _grid(call, gx, gy, gz=0, *, jitter=0.1, tol=1e-8, rhs=1, fp32=False, skip=0.0, autotune=True):
    return {"call": call, "problem": "grid", "gx": gx, "gy": gy, "gz": gz, "jitter": jitter, "tol": tol, "rhs": rhs,
            "fp32": fp32, "skip": skip, "autotune": autotune}


def _graph(call, points, *, tol=1e-8, rhs=1, fp32=False, autotune=True):
    return {"call": call, "problem": "graph", "points": points, "tol": tol, "rhs": rhs, "fp32": fp32, "skip": 0.0,
            "autotune": autotune}


def _group(problems, rhs, n_lo, n_hi):
    return {"call": "group", "problem": "grids", "problems": problems, "rhs": rhs, "n_lo": n_lo, "n_hi": n_hi,
            "tol": 1e-8}


def listed():
    return [
        # one preconditioner application on a tiny problem: nothing but launches and latency
        dict(_grid("kcycle", 33, 31), name="kcycle 2d 33x31"),
        # a small problem solved again and again with new right-hand sides
        dict(_grid("solve", 45, 45), name="solve 2d 45x45"),
        # a new small 2D problem with odd sides, as the serving loop's smaller requests
        dict(_grid("setup_solve", 181, 173, autotune=False), name="setup+solve 2d 181x173"),
        # a new small 3D problem with three different sides
        dict(_grid("setup_solve", 41, 37, 29, autotune=False), name="setup+solve 3d 41x37x29"),
        # the benchmark's workload: 128^3, FP64, tol 1e-8
        dict(_grid("setup_solve", 128, 128, 128), name="setup+solve 3d 128"),
        # the same with level skipping below coarsening ratio 2, as the benchmark also reports
        dict(_grid("setup_solve", 128, 128, 128, skip=2.0), name="setup+solve 3d 128 skip"),
        # a kept 2D hierarchy of a million unknowns, sides that no tile divides
        dict(_grid("solve", 1003, 997), name="solve 2d 1003x997"),
        # a served request on a resident problem: a batch of 8 in the mixed precision mode
        dict(_grid("solve", 100, 100, 100, rhs=8, fp32=True, autotune=False), name="batch 8 fp32 3d 100"),
        # an irregular graph with rows of very different lengths, new matrix, FP64
        dict(_graph("setup_solve", 150000), name="setup+solve graph 150k"),
        # many right-hand sides on a kept graph hierarchy, mixed precision
        dict(_graph("solve", 300000, rhs=8, fp32=True), name="batch 8 fp32 graph 300k"),
        # 16 small problems x 4 right-hand sides in one launch
        dict(_group(16, 4, 500, 8000), name="group 16x4"),
        # the largest benchmark: 256^3, unit weights, tol 1e-10
        dict(_grid("setup_solve", 256, 256, 256, jitter=0.0, tol=1e-10), name="setup+solve 3d 256"),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def draw(rng):
    """A case with sizes log-uniform over the range of its call."""
    call = rng.choice(["kcycle", "solve", "setup_solve", "setup_kcycle", "batch", "graph", "graph_batch", "group"])
    if call == "group":
        lo = rng.randrange(500, 2000)
        return _group(rng.randrange(2, 24), rng.randrange(1, 5), lo, rng.randrange(2 * lo, 9000))
    if call == "graph":
        return _graph(rng.choice(["setup_solve", "setup_kcycle", "solve"]), int(_log(rng, 2000, 300000)))
    if call == "graph_batch":
        return _graph("solve", int(_log(rng, 2000, 300000)), rhs=rng.randrange(2, 9), fp32=rng.random() < 0.5)
    three = rng.random() < 0.6
    n = _log(rng, 1000, 4e6 if three else 2e6)
    d = 3 if three else 2
    side = n ** (1.0 / d)
    sides = [max(3, int(round(side * rng.uniform(0.8, 1.25)))) for _ in range(d)]
    skip = 2.0 if rng.random() < 0.2 else 0.0
    autotune = rng.random() < 0.5
    if call == "batch":
        return _grid("solve", *sides, rhs=rng.randrange(2, 9) if n < 1e6 else 2, fp32=rng.random() < 0.5, skip=skip,
                     autotune=autotune)
    # the preconditioner alone stays in FP64: in the mixed mode its result is FP32 data
    fp32 = "solve" in call and rng.random() < 0.3
    return _grid(call, *sides, fp32=fp32, skip=skip, autotune=autotune)


def _dims(case):
    return tuple(v for v in (case["gx"], case["gy"], case["gz"]) if v)


def _matrix(case, seed):
    """The case's CSR matrix on the GPU, from the seed."""
    if case["problem"] == "grid":
        return amg.device_grid_laplacian(_dims(case), case["jitter"], seed)
    rp, ci, va = inputs.rgg_laplacian(case["points"], seed=seed, weight_range=(0.5, 1.5))
    return tuple(torch.from_numpy(v).cuda() for v in (rp, ci, va))


def _rhs(n, count, seed):
    b = torch.empty((count, n), dtype=torch.float64, device="cuda")
    for k in range(count):
        amg.device_rhs(b[k], 64 * seed + k)
    return b


def _group_problems(case, seed):
    """Dimensions and matrix seed of each problem of a group."""
    got = []
    lo, hi = math.log(case["n_lo"]), math.log(case["n_hi"])
    for k in range(case["problems"]):
        u = inputs.uniform(91, [2 * k, 2 * k + 1])  # the shapes belong to the case, the values to the seed
        d = 2 if u[0] < 0.5 else 3
        side = max(3, int(round(math.exp(lo + u[1] * (hi - lo)) ** (1.0 / d))))
        got.append(((side,) * (d - 1) + (side + 1,), 1000 * seed + k))
    return got


def _options(case):
    return {"max_rhs": case["rhs"], "precision": FP32 if case["fp32"] else amg.AMG_PREC_FP64,
            "skip_ratio": case["skip"], "autotune": int(case["autotune"])}


def prepare(case, seed):
    if case["call"] == "group":
        jobs = []
        for dims, s in _group_problems(case, seed):
            h = amg.Hierarchy(*amg.device_grid_laplacian(dims, 0.1, s), max_rhs=case["rhs"], autotune=0)
            b = _rhs(h.n, case["rhs"], s)
            x = torch.zeros_like(b)
            jobs += [(h, c, b[c], x[c]) for c in range(case["rhs"])]
        return {"call": "group", "jobs": jobs, "tol": case["tol"]}
    csr = _matrix(case, seed)
    b = _rhs(csr[0].numel() - 1, case["rhs"], seed)
    state = {"call": case["call"], "b": b, "x": torch.zeros_like(b), "tol": case["tol"], "options": _options(case)}
    if case["call"].startswith("setup"):
        state["csr"] = csr
    else:
        state["h"] = amg.Hierarchy(*csr, **state["options"])
    return state


def _solve(h, s):
    s["x"].zero_()  # the initial guess
    if s["b"].shape[0] == 1:
        h.solve(s["b"][0], s["x"][0], s["tol"])
    else:
        h.solve_batch(s["b"], s["x"], s["tol"])
    return s["x"]


def run(state):
    call = state["call"]
    if call == "group":
        for _, _, _, x in state["jobs"]:
            x.zero_()
        amg.solve_group(state["jobs"], state["tol"])
        return torch.cat([x for _, _, _, x in state["jobs"]])
    if call == "solve":
        return _solve(state["h"], state)
    if call == "kcycle":
        state["h"].kcycle(state["b"][0], state["x"][0])
        return state["x"]
    with amg.Hierarchy(*state["csr"], **state["options"]) as h:
        levels = np.zeros((MAX_LEVELS, 2), np.int64)  # unknowns and stored entries of each level
        for k in range(h.num_levels):
            levels[k] = h.level_sizes(k)[:2]
        if call == "setup_solve":
            _solve(h, state)
        else:
            h.kcycle(state["b"][0], state["x"][0])
    return {"x": state["x"], "levels": levels}


def _entries(dims):
    n = math.prod(dims)
    return n + sum(2 * (n - n // d) for d in dims)


def work(case):
    """Matrix and right-hand sides read once, solutions written once; one product with
    the matrix per right-hand side."""
    if case["call"] == "group":
        sizes = [(math.prod(d), _entries(d)) for d, _ in _group_problems(case, 1)]
    elif case["problem"] == "grid":
        sizes = [(math.prod(_dims(case)), _entries(_dims(case)))]
    else:
        sizes = [(case["points"], 9 * case["points"])]
    rhs = case["rhs"]
    return {"bytes": sum(12 * nnz + 4 * (n + 1) + 16 * n * rhs for n, nnz in sizes),
            "flops": sum(2 * nnz * rhs for _, nnz in sizes)}


def _conjugate_gradients(csr, b):
    """A x = b for the rows of b by Jacobi-preconditioned conjugate gradients in FP64,
    continued from the true residual until it stops falling."""
    rp, ci, va = csr
    n = rp.numel() - 1
    a = torch.sparse_csr_tensor(rp, ci, va, size=(n, n))
    rows = torch.repeat_interleave(torch.arange(n, device=rp.device), (rp[1:] - rp[:-1]).long())
    diag = va[rows == ci].unsqueeze(1)
    f = b.t().contiguous()
    x = torch.zeros_like(f)
    norm = f.norm(dim=0)
    for _ in range(3):
        r = f - a @ x
        first = r.norm(dim=0).clamp_min(1e-300)
        z = r / diag
        p = z.clone()
        rz = (r * z).sum(0)
        for k in range(20000):
            q = a @ p
            alpha = rz / (p * q).sum(0).clamp_min(1e-300)
            x += alpha * p
            r -= alpha * q
            z = r / diag
            rz, old = (r * z).sum(0), rz
            p = z + (rz / old.clamp_min(1e-300)) * p
            if k % 25 == 24 and bool((r.norm(dim=0) <= 1e-13 * torch.minimum(first, norm)).all()):
                break
        if bool(((f - a @ x).norm(dim=0) <= 1e-15 * norm).all()):
            break
    return x.t().contiguous()


def exact(case, seed):
    """The solutions of the linear systems (a preconditioner application has no value of
    its own: it is what the hierarchy makes it)."""
    if case["call"].endswith("kcycle"):
        return None
    if case["call"] == "group":
        out = []
        for dims, s in _group_problems(case, seed):
            csr = amg.device_grid_laplacian(dims, 0.1, s)
            out.append(_conjugate_gradients(csr, _rhs(math.prod(dims), case["rhs"], s)).reshape(-1))
        return torch.cat(out)
    csr = _matrix(case, seed)
    x = _conjugate_gradients(csr, _rhs(csr[0].numel() - 1, case["rhs"], seed))
    return x if case["call"] == "solve" else {"x": x, "levels": None}
