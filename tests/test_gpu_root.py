"""Root step: sums over groups of scenarios (each its own up to 32), root sizes at the edges
of the 16 x 16 tiles, the root factored with the first solve's root step and alone, and the
info of a factorization that fails, then succeeds, on one plan.  Reference: the FP64 oracle at
the parity suite's 1e-11."""
import numpy as np
import pytest

from oracle import oracle
from synth.branch_system import make_system

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


@pytest.mark.parametrize("S", [1, 31, 32, 33, 70])
@pytest.mark.parametrize("n,nrhs", [(3, 1), (16, 8), (16, 9), (17, 2), (32, 1), (33, 1), (48, 3),
                                    (49, 1), (64, 2)])
def test_root_sizes(S, n, nrhs):
    from paper_2609_29977_amd import bmpc
    s = make_system(S, 3, n, nrhs, 1e-2, 10 + S)
    ref, info = oracle.solve(s.D, s.E, s.C, s.R, s.b, nthreads=8)
    assert info == 0
    K = tuple(_dev(a) for a in (s.D, s.E, s.C, s.R))
    b = _dev(s.b)
    p = bmpc.Plan(S, 3, n, nrhs, "fp64")
    xs = [p.factor_solve(*K, b)]
    p.factor(*K)
    xs.append(p.solve(b))
    assert p.info() == 0
    for x in xs:
        assert float(np.max(np.abs(x.cpu().numpy() - ref))) <= 1e-11 * np.max(np.abs(ref))
    p.close()


@pytest.mark.parametrize("fused", [True, False])
@pytest.mark.parametrize("n", [8, 16, 24, 40])
def test_info_of_each_factorization(n, fused):
    from paper_2609_29977_amd import bmpc
    S, N = 5, 6
    s = make_system(S, N, n, 1, 1e-2, 3)
    good = [_dev(a) for a in (s.D, s.E, s.C, s.R)]
    b = _dev(s.b)
    p = bmpc.Plan(S, N, n, 1, "fp64")

    def info(K):
        p.factor_solve(*K, b) if fused else p.factor(*K)
        return p.info()

    D = s.D.copy()
    D[3, 2, n - 1, n - 1] = -1e6  # a tail block: scenario 3, stage 2
    bad_tail = [_dev(D), *good[1:]]
    R = s.R.copy()
    R[n - 1, n - 1] = -1e6
    bad_root = [*good[:3], _dev(R)]
    tail, root = (3 * N + 2) * n + n, S * N * n + n
    assert [info(K) for K in (good, bad_tail, good, bad_root, good, bad_tail, bad_root)] == \
        [0, tail, 0, root, 0, tail, root]
    p.close()
