"""Solves as matrix products over the right-hand sides: row tiles of 16 (n of 1..64, with and
without 16-byte rows), one to more than sixteen right-hand sides, levels whose pulls one or
several waves share; one right-hand side of padded blocks (row reads backward, merged top
levels); the same in a ragged batch.  Reference: the FP64 oracle, tolerances of the parity
suite (1e-11 FP64, 1e-10 FP32 with refinement); a ragged batch is bitwise its systems'
plans."""
import numpy as np
import pytest

from oracle import oracle
from synth.branch_system import make_system

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


SIZES = [(1, 3), (3, 1), (8, 2), (13, 1), (15, 16), (16, 9), (17, 1), (21, 5), (24, 1), (24, 12),
         (31, 1), (32, 17), (33, 1), (36, 16), (47, 2), (48, 18), (50, 1), (64, 1), (64, 16)]


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32", 1e-10)])
@pytest.mark.parametrize("n,nrhs", SIZES)
def test_against_the_oracle(n, nrhs, precision, tol):
    from paper_2609_29977_amd import bmpc
    S = 3
    for N in (1, 2, 6, 39, 70):  # levels 0, 1, 3, 6 (two and three waves), 7
        s = make_system(S, N, n, nrhs, 1e-2, 40 + N)
        ref, info = oracle.solve(s.D, s.E, s.C, s.R, s.b, nthreads=8)
        assert info == 0
        K = (_dev(s.D), _dev(s.E) if N > 1 else None, _dev(s.C), _dev(s.R))
        b = _dev(s.b)
        p = bmpc.Plan(S, N, n, nrhs, precision)
        if precision == "fp64":
            xs = [p.factor_solve(*K, b)]
            p.factor(*K)
            xs.append(p.solve(b))
        else:
            xs = [p.factor_refine(*K, b, tol=1e-13, max_iters=10)]
        assert p.info() == 0
        for x in xs:
            err = float(np.max(np.abs(x.cpu().numpy() - ref)) / np.max(np.abs(ref)))
            assert err <= tol, (N, err)
        p.close()


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nrhs", [1, 8, 17])
def test_ragged_is_bitwise_its_plans(nrhs, precision):
    import torch

    from paper_2609_29977_amd import bmpc
    shapes = [(5, 70, 32), (3, 33, 24), (2, 9, 21), (4, 40, 13), (3, 20, 16), (6, 64, 8),
              (2, 2, 20), (3, 1, 31), (2, 130, 12), (3, 15, 5)]
    systems = [make_system(S, N, n, nrhs, 1e-2, 70 + i) for i, (S, N, n) in enumerate(shapes)]
    rp = bmpc.RaggedPlan([(S, N, n, nrhs) for S, N, n in shapes], precision)
    parts = lambda name: [_dev(getattr(s, name)) for s in systems]
    K = (rp.pack(0, parts("D")), rp.pack(1, [_dev(s.E) if s.N > 1 else None for s in systems]),
         rp.pack(2, parts("C")), rp.pack(3, parts("R")))
    b = rp.pack(4, parts("b"))

    def run(p, K, b):
        if precision == "fp64":
            out = [p.factor_solve(*K, b)]
            p.factor(*K)
            return out + [p.solve(b)]
        return [p.factor_refine(*K, b, tol=0.0, max_iters=2)]

    xs = run(rp, K, b)
    for i, s in enumerate(systems):
        p = bmpc.Plan(s.S, s.N, s.n, nrhs, precision)
        own = run(p, (_dev(s.D), _dev(s.E) if s.N > 1 else None, _dev(s.C), _dev(s.R)), _dev(s.b))
        for x, xi in zip(xs, own):
            assert torch.equal(rp.unpack(4, x, i), xi.reshape(-1)), (i, shapes[i])
        p.close()
    rp.close()
