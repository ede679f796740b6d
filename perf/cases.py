"""The work that a program using this library has it do, as timed cases.

Every case goes through the public entry points (bmpc.Plan, bmpc.RaggedPlan,
bmpc.assemble_qp, autograd) on seeded inputs made on the GPU: the recipe of the
benchmark's systems (E and C entries 0.5 N(0, 1/n), D = M M^T / n plus a multiple of the
identity that bounds the spectral norms of the row's couplings, R likewise), and for the
QP a synthetic linear branch-MPC problem.

Kinds of a case:
  factor_solve   FP64 factor and solve in one call (one Newton system, one answer)
  factor+solve   FP64, the two calls one after the other (the factor is kept)
  solve          FP64 solves with a kept factor (ADMM, simulation, sensitivities)
  refine         FP32 factor with FP64-residual refinement in one call
  ragged         many systems of different shapes in one plan, FP32 with refinement
  grad           forward and backward of a batch of systems through autograd
  qp             IPM step: assembly of the reduced system, FP32 factor, refined solve
"""
import random

import torch

from paper_2609_29977_amd import autograd, bmpc

F64 = torch.float64
DEV = "cuda"


def listed():
    return [
        # the smallest system of the test suite: launches and host calls are all it costs
        {"name": "tiny_fp64", "kind": "factor_solve", "S": 4, "N": 16, "n": 8, "nrhs": 1},
        # a quadrotor-sized controller at its control rate: 20 scenarios, 30 stages, n = 16
        {"name": "mpc_small_fp64", "kind": "factor_solve", "S": 20, "N": 30, "n": 16, "nrhs": 1},
        # the large end of the same grid, factor and solve as separate calls
        {"name": "mpc_long_fp64", "kind": "factor+solve", "S": 100, "N": 160, "n": 16, "nrhs": 1},
        # the parity workload in mixed precision, four right-hand sides, to a tolerance
        {"name": "mid_fp32_4rhs", "kind": "refine", "S": 256, "N": 128, "n": 16, "nrhs": 4,
         "tol": 1e-12, "iters": 10, "stop": "correction"},
        # the benchmark's system in mixed precision, one correction
        {"name": "big_fp32", "kind": "refine", "S": 512, "N": 256, "n": 32, "nrhs": 1,
         "tol": 0.0, "iters": 1, "stop": "correction"},
        # the benchmark's system in FP64
        {"name": "big_fp64", "kind": "factor_solve", "S": 512, "N": 256, "n": 32, "nrhs": 1},
        # a block size that is no tile (padded blocks), an odd scenario count
        {"name": "odd_fp64", "kind": "factor_solve", "S": 73, "N": 100, "n": 24, "nrhs": 1},
        # blocks beyond one 32 x 32 tile (larger vehicles, condensed stages)
        {"name": "block48_fp64", "kind": "factor_solve", "S": 64, "N": 64, "n": 48, "nrhs": 1},
        # sensitivities: a kept factor and a dozen right-hand sides at once
        {"name": "resolve_fp64_12rhs", "kind": "solve", "S": 128, "N": 128, "n": 32, "nrhs": 12},
        # a server's batch of different problems in one ragged plan
        {"name": "ragged_fp32", "kind": "ragged", "systems": 64, "shape_seed": 1, "nrhs": 1},
        # training through the solve: 64 systems, forward and backward
        {"name": "grad_fp64", "kind": "grad", "B": 64, "S": 128, "N": 64, "n": 16, "nrhs": 1},
        # one interior-point step from the QP's data
        {"name": "ipm_step", "kind": "qp", "S": 256, "N": 128, "nx": 12, "nu": 4},
    ]


def _log(rng, lo, hi):
    return max(lo, min(hi, round(lo * (hi / lo) ** rng.random())))


def draw(rng):
    kind = rng.choice(["factor_solve", "factor_solve", "factor+solve", "solve", "refine",
                       "refine", "ragged", "grad", "qp"])
    if kind == "ragged":
        return {"kind": kind, "systems": _log(rng, 4, 64), "shape_seed": rng.randrange(2, 10 ** 6),
                "nrhs": rng.choice([1, 1, 1, 2, 3])}
    if kind == "qp":
        nu = rng.randint(1, 8)
        nx = rng.randint(4, 32 - nu)
        while True:
            S, N = _log(rng, 4, 256), _log(rng, 8, 128)
            if S * N * (nx + nu) ** 2 <= 256 * 128 * 256:
                return {"kind": kind, "S": S, "N": N, "nx": nx, "nu": nu}
    # block sizes: the tiles, and everything in between
    n = rng.choice([8, 16, 16, 32, 32, rng.randint(4, 32), rng.randint(4, 32), rng.randint(33, 64)])
    if kind == "grad":
        n = min(n, 32)
        while True:
            B, S, N = _log(rng, 1, 64), _log(rng, 4, 128), _log(rng, 4, 64)
            if B * S * N * n * n <= 64 * 128 * 64 * 256:
                return {"kind": kind, "B": B, "S": S, "N": N, "n": n, "nrhs": rng.choice([1, 1, 2])}
    nrhs = rng.choice([1, 1, 1, 2, 4, 9, 16]) if kind == "solve" else rng.choice([1, 1, 1, 2, 4])
    while True:
        S, N = _log(rng, 2, 512), _log(rng, 2, 256)
        if S * N * n * n * max(1, nrhs) <= 512 * 256 * 1024 // (8 if n > 32 else 2):
            break
    case = {"kind": kind, "S": S, "N": N, "n": n, "nrhs": nrhs}
    if kind == "refine":
        case.update(rng.choice([{"tol": 0.0, "iters": 1, "stop": "correction"},
                                {"tol": 1e-12, "iters": 10, "stop": "correction"},
                                {"tol": 2e-15, "iters": 10, "stop": "backward_error"}]))
    return case


# ---- inputs ------------------------------------------------------------------------


def _norm_bound(A):
    """An upper bound of the spectral norm of every block, close to it: the Frobenius norm
    of (A^T A)^4 to the power 1/8."""
    P = A.mT.contiguous() @ A
    P = P @ P
    P = P @ P
    return torch.linalg.matrix_norm(P) ** 0.125


def _systems(B, S, N, n, nrhs, delta, seed):
    """D, E, C, R, b of B stacked systems."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kw = dict(dtype=F64, device=DEV, generator=g)
    E = torch.randn((B, S, N - 1, n, n), **kw).mul_(0.5 / n ** 0.5)
    C = torch.randn((B, S, n, n), **kw).mul_(0.5 / n ** 0.5)
    M = torch.randn((B, S, N, n, n), **kw)
    MR = torch.randn((B, n, n), **kw)
    b = torch.randn((B, nrhs, (S * N + 1) * n), **kw)
    D = (M @ M.mT.contiguous()).div_(n)
    del M
    shift = torch.full((B, S, N), float(delta), dtype=F64, device=DEV)
    if N > 1:
        e = _norm_bound(E)
        shift[..., 1:] += e
        shift[..., :-1] += e
    c = _norm_bound(C)
    shift[..., 0] += c
    D.diagonal(dim1=-2, dim2=-1).add_(shift[..., None])
    D = (D + D.mT) * 0.5
    R = MR @ MR.mT.contiguous() / n
    R.diagonal(dim1=-2, dim2=-1).add_((c.sum(-1) + delta)[:, None])
    R = (R + R.mT) * 0.5
    return D, E, C, R, b


def _one(case, seed):
    D, E, C, R, b = _systems(1, case["S"], case["N"], case["n"], case["nrhs"], 1e-2, seed)
    return D[0], E[0], C[0], R[0], b[0]


def _ragged_shapes(case):
    rng = random.Random(case["shape_seed"])
    return [(rng.randint(8, 256), rng.randint(16, 256), rng.choice([8, 16, 32]), case["nrhs"])
            for _ in range(case["systems"])]


def _ragged_systems(case, seed):
    for i, (S, N, n, nrhs) in enumerate(_ragged_shapes(case)):
        yield [t[0] for t in _systems(1, S, N, n, nrhs, 1e-2, seed * 1000 + i)]


QP_TAU, QP_DELTA = 1e-6, 1e-3


def _qp(case, seed):
    """Q, A, G, w per link and the right-hand side: per-scenario linear dynamics as
    equality rows, box constraints as inequality rows, interior-point weights spread over
    four decades."""
    S, N, nx, nu = case["S"], case["N"], case["nx"], case["nu"]
    n = nx + nu
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    kw = dict(dtype=F64, device=DEV, generator=g)
    eye = torch.eye(nx, dtype=F64, device=DEV)
    Ad = eye + 0.1 / nx ** 0.5 * torch.randn((nx, nx), **kw) + 0.02 * torch.randn((S, 1, nx, nx), **kw)
    Bd = 0.1 * torch.randn((nx, nu), **kw) + 0.02 * torch.randn((S, 1, nx, nu), **kw)
    M = torch.randn((S, N + 1, 2 * n, 2 * n), **kw)
    Q = (M @ M.mT.contiguous()).div_(2 * n)
    Q = (Q + Q.mT) * 0.5
    Q[:, N, n:, :] = 0.0
    Q[:, N, :, n:] = 0.0
    A = torch.zeros((S, N + 1, nx, 2 * n), dtype=F64, device=DEV)
    A[:, :N, :, :nx] = Ad
    A[:, :N, :, nx:n] = Bd
    A[:, :N, :, n:n + nx] = -eye
    G = torch.zeros((S, N + 1, 2 * n, 2 * n), dtype=F64, device=DEV)
    I = torch.eye(n, dtype=F64, device=DEV)
    G[:, :N, :n, n:] = I
    G[:, :N, n:, n:] = -I
    w = 10.0 ** (torch.rand((S, N + 1, 2 * n), **kw) * 4 - 3)
    w[:, N] = 1.0
    b = torch.randn((1, (S * N + 1) * n), **kw)
    return Q, A, G, w, b


def prepare(case, seed):
    kind = case["kind"]
    if kind == "ragged":
        plan = bmpc.RaggedPlan(_ragged_shapes(case), "fp32")
        parts = list(zip(*_ragged_systems(case, seed)))
        D, E, C, R, b = (plan.pack(i, p) for i, p in enumerate(parts))
        return {"kind": kind, "plan": plan, "K": (D, E, C, R), "b": b, "x": torch.zeros_like(b)}
    if kind == "grad":
        ins = _systems(case["B"], case["S"], case["N"], case["n"], case["nrhs"], 1e-2, seed)
        g = torch.Generator(device=DEV)
        g.manual_seed(seed + 1)
        gx = torch.randn(ins[4].shape, dtype=F64, device=DEV, generator=g)
        return {"kind": kind, "ins": [t.requires_grad_() for t in ins], "gx": gx}
    if kind == "qp":
        Q, A, G, w, b = _qp(case, seed)
        n = case["nx"] + case["nu"]
        S, N = case["S"], case["N"]
        out = tuple(torch.empty(s, dtype=F64, device=DEV)
                    for s in ((S, N, n, n), (S, N - 1, n, n), (S, n, n), (n, n)))
        return {"kind": kind, "plan": bmpc.Plan(S, N, n, 1, "fp32"), "qp": (Q, A, G, w),
                "K": out, "b": b, "x": torch.empty_like(b)}
    D, E, C, R, b = _one(case, seed)
    plan = bmpc.Plan(case["S"], case["N"], case["n"], case["nrhs"],
                     "fp32" if kind == "refine" else "fp64")
    st = {"kind": kind, "plan": plan, "K": (D, E, C, R), "b": b, "x": torch.empty_like(b)}
    if kind == "refine":
        plan.set_refine_stop(case["stop"])
        st["opt"] = {"tol": case["tol"], "max_iters": case["iters"]}
    elif kind == "solve":
        plan.factor(D, E, C, R)
    return st


# ---- the calls ---------------------------------------------------------------------


def run(st):
    kind = st["kind"]
    if kind == "factor_solve":
        return st["plan"].factor_solve(*st["K"], st["b"], st["x"])
    if kind == "factor+solve":
        st["plan"].factor(*st["K"])
        return st["plan"].solve(st["b"], st["x"])
    if kind == "solve":
        return st["plan"].solve(st["b"], st["x"])
    if kind == "refine":
        return st["plan"].factor_refine(*st["K"], st["b"], st["x"], **st["opt"])
    if kind == "ragged":
        return st["plan"].factor_refine(*st["K"], st["b"], st["x"], tol=0.0, max_iters=1)
    if kind == "grad":
        x = autograd.batched_branch_solve(*st["ins"], "fp64")
        return [x.detach(), *torch.autograd.grad(x, st["ins"], st["gx"])]
    bmpc.assemble_qp(*st["qp"], QP_TAU, QP_DELTA, out=st["K"])
    st["plan"].factor(*st["K"])
    st["plan"].refine(*st["K"], st["b"], st["x"], tol=1e-10, max_iters=10)
    return [*st["K"], st["x"]]


# ---- what a pass cannot do without -------------------------------------------------


def _work(S, N, n, nrhs, T, factor=True, solve=True):
    """Bytes: D and R as lower triangles, E, C, b and x once; the factor (T bytes an
    entry: L_jj lower, two blocks per chain position) written by a factorization, read by
    a solve that is given one.  Flops: block elimination, and the two sweeps."""
    tri, nn, m = n * (n + 1) // 2, n * n, N - 1
    L = S * (N * tri + (2 * m + 1) * nn)
    by = fl = 0.0
    if factor:
        by += 8.0 * (S * N * tri + S * m * nn + S * nn + tri) + T * L
        fl += S * (m * (n ** 3 / 3.0 + 2 * n ** 3 + 2 * n ** 3 + 2 * n ** 3) + 7 * n ** 3 / 3.0)
    elif solve:
        by += T * L
    if solve:
        by += 16.0 * nrhs * (S * N + 1) * n
        fl += nrhs * 4.0 * L
    return by, fl


def work(case):
    kind = case["kind"]
    if kind == "ragged":
        parts = [_work(S, N, n, q, 4) for S, N, n, q in _ragged_shapes(case)]
    elif kind == "grad":
        S, N, n, B, q = case["S"], case["N"], case["n"], case["B"], case["nrhs"]
        by, fl = _work(S, N, n, q, 8)
        len_ = (S * N + 1) * n
        out = 8.0 * (S * (2 * N) * n * n + n * n)  # dD, dE, dC, dR
        parts = [(B * (by + out + 16.0 * q * len_), B * (2 * fl + 8.0 * q * S * N * n * n))]
    elif kind == "qp":
        S, N, n = case["S"], case["N"], case["nx"] + case["nu"]
        by, fl = _work(S, N, n, 1, 4)
        rows, links = case["nx"] + 2 * n, S * (N + 1)
        read = 8.0 * links * (4 * n * n + rows * 2 * n + 2 * n)
        parts = [(read + by, fl + links * rows * 6.0 * n * n)]
    else:
        parts = [_work(case["S"], case["N"], case["n"], case["nrhs"],
                       4 if kind == "refine" else 8, kind != "solve", True)]
    return {"bytes": sum(p[0] for p in parts), "flops": sum(p[1] for p in parts)}


# ---- the same in plain torch, 64 bits ----------------------------------------------


def _exact_factor(D, E, C, R):
    """Block elimination of every tail from its last stage to its first, then the root."""
    S, N, n, _ = D.shape
    L, W = [None] * N, [None] * N
    A = D[:, N - 1].clone()
    for k in range(N - 1, -1, -1):
        L[k] = torch.linalg.cholesky(A)
        low = E[:, k - 1] if k > 0 else C.mT
        W[k] = torch.linalg.solve_triangular(L[k], low.contiguous(), upper=False)
        if k > 0:
            A = D[:, k - 1] - W[k].mT.contiguous() @ W[k]
    root = torch.linalg.cholesky(R - (W[0].mT.contiguous() @ W[0]).sum(0))
    return L, W, root


def _exact_solve(F, S, N, n, b):
    """x of b [nrhs][len] with the factor F."""
    L, W, root = F
    q = b.shape[0]
    t = b[:, :S * N * n].reshape(q, S, N, n).permute(1, 2, 3, 0).contiguous()  # S N n q
    r0 = b[:, S * N * n:].T.contiguous()
    y = [None] * N
    v = t[:, N - 1]
    for k in range(N - 1, -1, -1):
        y[k] = torch.linalg.solve_triangular(L[k], v.contiguous(), upper=False)
        push = W[k].mT.contiguous() @ y[k]
        if k > 0:
            v = t[:, k - 1] - push
        else:
            r0 = r0 - push.sum(0)
    z = torch.linalg.solve_triangular(root, r0, upper=False)
    x0 = torch.linalg.solve_triangular(root.mT, z, upper=True)
    prev = x0.expand(S, n, q)
    out = torch.empty_like(t)
    for k in range(N):
        v = y[k] - W[k] @ prev.contiguous()
        prev = torch.linalg.solve_triangular(L[k].mT, v, upper=True)
        out[:, k] = prev
    return torch.cat([out.permute(3, 0, 1, 2).reshape(q, -1), x0.T], 1)


def _exact_system(D, E, C, R, *vectors):
    S, N, n, _ = D.shape
    F = _exact_factor(D, E, C, R)
    return [_exact_solve(F, S, N, n, b) for b in vectors]


def _exact_grad(case, seed):
    st = prepare(case, seed)
    S, N, n, q = case["S"], case["N"], case["n"], case["nrhs"]
    D, E, C, R, b = (t.detach() for t in st["ins"])
    outs = []
    for i in range(case["B"]):
        x, lam = _exact_system(D[i], E[i], C[i], R[i], b[i], st["gx"][i])

        def split(v):
            return v[:, :S * N * n].reshape(q, S, N, n), v[:, S * N * n:].reshape(q, n)

        (xt, xr), (lt, lr) = split(x), split(lam)

        def outer(u, v):
            return (u[..., :, None] * v[..., None, :]).sum(0)

        dD, dR = outer(lt, xt), outer(lr, xr)
        outs.append((x, -(dD + dD.mT) / 2,
                     -(outer(lt[:, :, 1:], xt[:, :, :-1]) + outer(xt[:, :, 1:], lt[:, :, :-1])),
                     -(outer(lr[:, None].expand(q, S, n), xt[:, :, 0])
                       + outer(xr[:, None].expand(q, S, n), lt[:, :, 0])),
                     -(dR + dR.mT) / 2, lam))
    return [torch.stack(t) for t in zip(*outs)]


def exact(case, seed):
    kind = case["kind"]
    if kind == "ragged":
        return torch.cat([_exact_system(*s)[0].reshape(-1) for s in _ragged_systems(case, seed)])
    if kind == "grad":
        return _exact_grad(case, seed)
    if kind == "qp":
        Q, A, G, w, b = _qp(case, seed)
        n, N = case["nx"] + case["nu"], case["N"]
        X = torch.cat([A / QP_DELTA ** 0.5, G / (w + QP_DELTA).sqrt()[..., None]], 2)
        M = Q + X.mT.contiguous() @ X
        I = torch.eye(n, dtype=F64, device=DEV)
        D = QP_TAU * I + M[:, :N, n:, n:] + M[:, 1:, :n, :n]
        E, C = M[:, 1:N, n:, :n].contiguous(), M[:, 0, :n, n:].contiguous()
        R = QP_TAU * I + M[:, 0, :n, :n].sum(0)
        return [D, E, C, R, *_exact_system(D, E, C, R, b)]
    D, E, C, R, b = _one(case, seed)
    return _exact_system(D, E, C, R, b)[0]
