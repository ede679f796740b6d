"""Rounding error of the FP64 solves: many right-hand sides at once (matrix products) do no worse
than the same right-hand sides one at a time (partial sums of a block's registers), against a
reference refined in extended precision.  Both take the same operations and differ in the order
of their sums alone, so their root mean square errors agree but for the spread of a sample: over 8
systems of 12 right-hand sides less than 8 %."""
import numpy as np
import pytest

from synth.branch_system import make_system

pytestmark = pytest.mark.gpu


def _dense(s):
    S, N, n = s.S, s.N, s.n
    sym = lambda a: np.tril(a) + np.tril(a, -1).T
    r0 = S * N * n
    K = np.zeros((r0 + n, r0 + n))
    for i in range(S):
        for k in range(N):
            a = (i * N + k) * n
            K[a:a + n, a:a + n] = sym(s.D[i, k])
            if k + 1 < N:
                K[a + n:a + 2 * n, a:a + n] = s.E[i, k]
                K[a:a + n, a + n:a + 2 * n] = s.E[i, k].T
        a = i * N * n
        K[r0:, a:a + n] = s.C[i]
        K[a:a + n, r0:] = s.C[i].T
    K[r0:, r0:] = sym(s.R)
    return K


def _extended(s):
    K = _dense(s)
    Kl, bl = K.astype(np.longdouble), s.b.T.astype(np.longdouble)
    x = np.linalg.solve(K, s.b.T).astype(np.longdouble)
    for _ in range(3):
        x = x + np.linalg.solve(K, (bl - Kl @ x).astype(np.float64))
    return x.T


def test_products_round_no_worse_than_registers():
    import torch
    from paper_2609_29977_amd import bmpc
    dev = lambda a: torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
    S, N, n, nrhs = 2, 8, 64, 12
    many, one = [], []
    for seed in range(8):
        s = make_system(S, N, n, nrhs, 1e-2, 1000 + seed)
        ref = _extended(s)
        p = bmpc.Plan(S, N, n, nrhs, "fp64")
        p.factor(dev(s.D), dev(s.E), dev(s.C), dev(s.R))
        x = p.solve(dev(s.b)).cpu().numpy()
        q = bmpc.Plan(S, N, n, 1, "fp64")
        q.factor(dev(s.D), dev(s.E), dev(s.C), dev(s.R))
        y = np.concatenate([q.solve(dev(s.b[r:r + 1])).cpu().numpy() for r in range(nrhs)])
        p.close()
        q.close()
        scale = np.max(np.abs(ref))
        many.append(np.mean(((x - ref) / scale) ** 2))
        one.append(np.mean(((y - ref) / scale) ** 2))
    many, one = (float(np.sqrt(np.mean(e))) for e in (many, one))
    assert many <= 1.08 * one, (many, one)
