"""Performance cases of the tiled Cholesky library: what its users have it do.

Six kinds of work, each through the public Python entry points:

  single  chol_factor of one matrix (a schedule, a tile side), then chol_solve
          of nrhs right-hand sides when nrhs > 0;
  solve   chol_solve against a factor the program already holds;
  batch   chol_factor_solve_batched: many matrices of uneven orders, one
          right-hand side each, in place;
  batch_refined
          chol_factor_solve_batched_mixed: the originals are kept, FP32 or
          FP64 trailing products, FP64 refinement in the same launch;
  refine  chol_factor_mixed (FP32 or BF16 trailing products) followed by
          chol_solve_refine (iterative refinement or PCG) to 1e-12;
  serve   a burst of factor + solve requests to the continuous-batching
          server, submitted together and all waited for.

Matrices are the repository's two recipes: the squared-exponential kernel on
points in the unit square (lengthscale 0.1, nugget 1e-2) and G G^T / n + I.
The factorizations work in place, so a pass first copies the kept original
into the working buffer, as a program that needs A again does.
"""
from __future__ import annotations

import math
import weakref

import numpy as np
import torch

from paper_2606_11937_amd import inputs
from paper_2606_11937_amd import tilechol as tc

TOL = 1e-12  # backward error asked of refined and served solutions


def listed():
    return [
        # the smallest call: one Gaussian process on 100 points, one tile
        {"name": "single_100", "kind": "single", "matrix": "se", "n": 100, "T": 128, "sched": "fork_join_lookahead",
         "nrhs": 1},
        # the parity configuration of the tests, plain fork-join, factor only
        {"name": "single_1024", "kind": "single", "matrix": "gg", "n": 1024, "T": 128, "sched": "fork_join",
         "nrhs": 0},
        # an ordinary Gaussian process with an odd order, the default tile side
        {"name": "single_3001", "kind": "single", "matrix": "se", "n": 3001, "T": 128, "sched": "fork_join_lookahead",
         "nrhs": 2},
        # the asynchronous task schedule at the middle of its benchmark sweep
        {"name": "single_8192_async", "kind": "single", "matrix": "se", "n": 8192, "T": 512, "sched": "async_dag",
         "nrhs": 0},
        # the benchmark's own step: n = 32768, T = 1024, factor + one solve
        {"name": "single_32768", "kind": "single", "matrix": "se", "n": 32768, "T": 1024,
         "sched": "fork_join_lookahead", "nrhs": 1},
        # predictions with a factor at hand: one vector, then many
        {"name": "solve_1500", "kind": "solve", "matrix": "se", "n": 1500, "T": 128, "nrhs": 1},
        {"name": "solve_8192x16", "kind": "solve", "matrix": "se", "n": 8192, "T": 128, "nrhs": 16},
        # many small systems at once (local models), then the benchmark's batch
        {"name": "batch_1000", "kind": "batch", "count": 1000, "lo": 32, "hi": 256},
        {"name": "batch_4096", "kind": "batch", "count": 4096, "lo": 32, "hi": 2048},
        # a batch whose originals are kept, FP32 products refined to 1e-12
        {"name": "batch_refined_512", "kind": "batch_refined", "count": 512, "lo": 64, "hi": 1024, "prec": "fp32"},
        # mixed precision at half the benchmark's order, its 16 right-hand sides
        {"name": "refine_16384", "kind": "refine", "matrix": "se", "n": 16384, "T": 1024, "nrhs": 16, "prec": "fp32",
         "method": "ir"},
        # a burst of requests to the server
        {"name": "serve_48", "kind": "serve", "count": 48, "lo": 64, "hi": 4096},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["single", "single", "solve", "batch", "batch_refined", "refine", "serve"])
    if kind == "single":
        n = _log_int(rng, 48, 16000)
        return {"kind": kind, "matrix": rng.choice(["se", "gg"]) if n <= 8192 else "se", "n": n,
                "T": rng.choice([128, 256, 512]) if n <= 8192 else rng.choice([512, 1024]),
                "sched": rng.choice(["fork_join_lookahead", "fork_join", "async_dag"]), "nrhs": rng.choice([0, 1, 2, 5])}
    if kind == "solve":
        return {"kind": kind, "matrix": "se", "n": _log_int(rng, 64, 16000), "T": 128, "nrhs": _log_int(rng, 1, 48)}
    if kind == "batch":
        return {"kind": kind, "count": _log_int(rng, 16, 1500), "lo": 32, "hi": _log_int(rng, 96, 1536)}
    if kind == "batch_refined":
        return {"kind": kind, "count": _log_int(rng, 16, 600), "lo": 32, "hi": _log_int(rng, 96, 1536),
                "prec": rng.choice(["fp32", "fp64"])}
    if kind == "refine":
        # BF16 products need a well-conditioned matrix, and PCG
        prec = rng.choice(["fp32", "fp32", "bf16"])
        n = _log_int(rng, 400, 16000 if prec == "fp32" else 8000)
        return {"kind": kind, "matrix": "se" if prec == "fp32" else "gg", "n": n,
                "T": rng.choice([256, 512]) if n <= 8192 else rng.choice([512, 1024]), "nrhs": _log_int(rng, 1, 24),
                "prec": prec, "method": "ir" if prec == "fp32" else "pcg"}
    return {"kind": kind, "count": _log_int(rng, 1, 64), "lo": 64, "hi": _log_int(rng, 128, 4096)}


# ------------------------------------------------------------------ inputs
def _gen(seed, salt):
    return torch.Generator(device="cuda").manual_seed(int(seed) * 1000003 + salt)


def _randn(seed, salt, *shape):
    return torch.randn(shape, generator=_gen(seed, salt), dtype=torch.float64, device="cuda")


def _matrix(case, seed):
    n = case["n"]
    if case["matrix"] == "se":
        return inputs.se_kernel_device(n, seed)
    G = _randn(seed, 1, n, n)
    A = G @ G.T / n
    A = (A + A.T) * 0.5
    A.diagonal().add_(1.0)
    return A


def _batch_orders(case, seed):
    """The orders are the case's own (every seed has the same work)."""
    return inputs.batch_sizes(case["count"], 3, case["lo"], case["hi"])


def _batch_views(flat, orders):
    out, at = [], 0
    for n in orders:
        out.append(flat[at:at + n * n].view(n, n))
        at += n * n
    return out


def _batch_inputs(case, seed):
    """One flat buffer of G G^T / n + I matrices and one of right-hand sides.
    G has 16 + n / 2 columns scaled to keep the spectrum of the recipe."""
    orders = _batch_orders(case, seed)
    flat = torch.empty(sum(n * n for n in orders), dtype=torch.float64, device="cuda")
    noise = _randn(seed, 1, max(orders) * (max(orders) // 2 + 16) + 4096 * 7)
    for i, (n, A) in enumerate(zip(orders, _batch_views(flat, orders))):
        k = n // 2 + 16
        at = (i * 7) % (4096 * 7)
        G = noise[at:at + n * k].view(n, k)
        torch.mm(G, G.T, out=A)
        A.mul_(1.0 / k)
        A.diagonal().add_(1.0)
    return orders, flat, _randn(seed, 2, sum(orders))


def _serve_requests(case, seed):
    orders = inputs.batch_sizes(case["count"], 4, case["lo"], case["hi"])
    rng = np.random.default_rng(int(seed) * 1000003 + 4)
    reqs = []
    for i, n in enumerate(orders):
        nrhs = 1 + i % tc.CHOL_SERVE_MAX_RHS
        reqs.append((rng.random((n, 2)), rng.standard_normal((n, nrhs)), float(rng.uniform(0.05, 0.5))))
    return reqs


class _State:
    pass


def prepare(case, seed):
    s = _State()
    s.kind = kind = case["kind"]
    if kind in ("single", "solve", "refine"):
        n, T, nrhs = case["n"], case["T"], case["nrhs"]
        s.T = T
        s.A = _matrix(case, seed)
        s.L = torch.empty_like(s.A)
        s.B = _randn(seed, 2, n, nrhs) if nrhs else None
        s.X = torch.empty_like(s.B) if nrhs else None
    if kind == "single":
        s.sched = case["sched"]
        s.fwork = tc.factor_workspace(n, T, s.sched)
        if nrhs:
            s.swork = torch.empty(tc.chol_solve_workspace_size(n, T, nrhs), dtype=torch.uint8, device="cuda")
    elif kind == "solve":
        s.L.copy_(s.A)
        tc.chol_factor(s.L, T, "fork_join")
        s.A = None
        s.swork = torch.empty(tc.chol_solve_workspace_size(n, T, nrhs), dtype=torch.uint8, device="cuda")
    elif kind == "refine":
        s.prec, s.method = case["prec"], case["method"]
        s.fwork = torch.empty(tc.chol_factor_mixed_workspace_size(n, T, s.prec), dtype=torch.uint8, device="cuda")
        s.rwork = torch.empty(tc.chol_refine_workspace_size(n, T, nrhs), dtype=torch.uint8, device="cuda")
    elif kind in ("batch", "batch_refined"):
        orders, s.flat, s.bflat = _batch_inputs(case, seed)
        s.lflat, s.xflat = torch.empty_like(s.flat), torch.empty_like(s.bflat)
        s.Ls, s.Xs = _batch_views(s.lflat, orders), list(torch.split(s.xflat, orders))
        if kind == "batch":
            nb = tc.chol_factor_solve_batched_workspace_size(orders)
        else:
            s.lflat.zero_()
            s.As, s.Bs = _batch_views(s.flat, orders), list(torch.split(s.bflat, orders))
            s.precs = [case["prec"]] * len(orders)
            nb = tc.chol_factor_solve_batched_mixed_workspace_size(orders, None, s.precs)
        s.work = torch.empty(nb, dtype=torch.uint8, device="cuda")
    else:
        s.requests = _serve_requests(case, seed)
        arena = torch.empty(max(2 << 30, sum(16 * len(p) ** 2 for p, _, _ in s.requests) + (512 << 20)),
                            dtype=torch.uint8, device="cuda")
        s.server = tc.Server(arena, pinned_bytes=256 << 20)
        weakref.finalize(s, s.server.close)
    return s


def run(s):
    if s.kind == "single":
        s.L.copy_(s.A)
        info = tc.chol_factor(s.L, s.T, s.sched, work=s.fwork)
        out = {"L": s.L, "info": info}
        if s.B is not None:
            s.X.copy_(s.B)
            tc.chol_solve(s.L, s.X, s.T, work=s.swork)
            out["X"] = s.X
        return out
    if s.kind == "solve":
        s.X.copy_(s.B)
        tc.chol_solve(s.L, s.X, s.T, work=s.swork)
        return s.X
    if s.kind == "refine":
        # the factor is the preconditioner; the result is the FP64 solution
        s.L.copy_(s.A)
        info = tc.chol_factor_mixed(s.L, s.T, s.prec, work=s.fwork)
        ok, _, _ = tc.chol_solve_refine(s.A, s.L, s.B, s.X, s.T, s.method, TOL, 60, work=s.rwork)
        return {"X": s.X, "info": info, "converged": ok}
    if s.kind == "batch":
        s.lflat.copy_(s.flat)
        s.xflat.copy_(s.bflat)
        infos = tc.chol_factor_solve_batched(s.Ls, s.Xs, work=s.work)
        return {"L": s.lflat, "X": s.xflat, "info": np.array(infos)}
    if s.kind == "batch_refined":
        infos, _, _ = tc.chol_factor_solve_batched_mixed(s.As, s.Ls, s.Bs, s.Xs, precs=s.precs, tol=TOL, work=s.work)
        return {"X": s.xflat, "info": np.array(infos)}
    ids = [s.server.submit(P, B, ell, 1e-2, TOL) for P, B, ell in s.requests]
    got = [s.server.wait(i) for i in ids]
    return {"X": np.concatenate([g[1].ravel() for g in got]), "status": np.array([g[0] for g in got])}


# -------------------------------------------------------------------- work
def _one(n, nrhs, factor=True, keep=True):
    """Bytes and flops of a factorization (lower triangle in, factor out) and
    a solve of nrhs right-hand sides (the factor read twice by a solve alone)."""
    tri = 8.0 * n * (n + 1) / 2
    b = (2 * tri if factor and keep else tri if factor else tri) + 16.0 * n * nrhs
    return b, (n ** 3 / 3.0 if factor else 0.0) + 2.0 * n * n * nrhs


def work(case):
    kind = case["kind"]
    if kind in ("single", "solve"):
        b, f = _one(case["n"], case["nrhs"], kind == "single")
    elif kind == "refine":
        # the low-precision factorization, and one FP64 residual pass over A
        b, f = _one(case["n"], case["nrhs"])
        b += 4.0 * case["n"] ** 2
        f += 2.0 * case["n"] ** 2 * case["nrhs"]
    elif kind == "serve":
        # the kernel matrices are formed on the device: only points, right-hand
        # sides and solutions cross the call
        b = f = 0.0
        for i, n in enumerate(inputs.batch_sizes(case["count"], 4, case["lo"], case["hi"])):
            nrhs = 1 + i % tc.CHOL_SERVE_MAX_RHS
            b += 16.0 * n * (1 + nrhs)
            f += n ** 3 / 3.0 + 2.0 * n * n * nrhs
    else:
        each = [_one(n, 1) for n in _batch_orders(case, 0)]
        b, f = sum(e[0] for e in each), sum(e[1] for e in each)
    return {"bytes": b, "flops": f}


# ------------------------------------------------------------------- exact
def _chol_solve(A, B):
    L = torch.linalg.cholesky(A)
    return L, torch.cholesky_solve(B, L) if B is not None else None


def exact(case, seed):
    kind = case["kind"]
    if kind in ("single", "solve", "refine"):
        A = _matrix(case, seed)
        B = _randn(seed, 2, case["n"], case["nrhs"]) if case["nrhs"] else None
        L, X = _chol_solve(A, B)
        if kind == "solve":
            return X
        if kind == "refine":
            return {"X": X, "info": None, "converged": None}
        L.add_(A.triu_(1))  # the strict upper triangle stays the input's
        out = {"L": L, "info": None}
        if X is not None:
            out["X"] = X
        return out
    if kind == "serve":
        xs = []
        for P, B, ell in _serve_requests(case, seed):
            p = torch.from_numpy(P).cuda()
            d = p[:, None, :] - p[None, :, :]
            A = torch.exp(-(d * d).sum(-1) / (2.0 * ell * ell))
            A.diagonal().add_(1e-2)
            xs.append(_chol_solve(A, torch.from_numpy(B).cuda())[1].cpu().numpy().ravel())
        return {"X": np.concatenate(xs), "status": None}
    orders, flat, bflat = _batch_inputs(case, seed)
    for A, b in zip(_batch_views(flat, orders), torch.split(bflat, orders)):
        L, x = _chol_solve(A, b[:, None])
        b.copy_(x[:, 0])
        if kind == "batch":
            A.triu_(1).add_(L)
    return {"L": flat if kind == "batch" else None, "X": bflat, "info": None}
