"""Factor passes of blocks up to 16 (windows walked level by level): chain lengths at the
edges of the windows (empty, one position, even and odd last positions, a left boundary
alone), every depth, padded blocks, one and the most fused right-hand sides, and launches
large enough for two waves per window at n <= 8.  Reference: the FP64 oracle; tolerances
are those of the parity suite (1e-11 FP64, 1e-10 FP32 with refinement)."""
import numpy as np
import pytest

from oracle import oracle
from synth.branch_system import make_system

pytestmark = pytest.mark.gpu


def _solve(S, N, n, nrhs, precision, wd, later=0):
    import torch

    from paper_2609_29977_amd import bmpc
    s = make_system(S, N, n, nrhs, 1e-2, 300 + N)
    ref, info = oracle.solve(s.D, s.E, s.C, s.R, s.b, nthreads=8)
    assert info == 0
    dev = lambda a: torch.from_numpy(a).to("cuda:0")
    K = (dev(s.D), dev(s.E) if N > 1 else None, dev(s.C), dev(s.R))
    b = dev(s.b)
    p = bmpc.Plan(S, N, n, nrhs, precision, wd, later_depth=later)
    if precision == "fp64":
        xs = [p.factor_solve(*K, b)]
        p.factor(*K)
        xs.append(p.solve(b))
    else:
        xs = [p.factor_refine(*K, b, tol=1e-13, max_iters=10)]
    assert p.info() == 0
    err = max(float(np.max(np.abs(x.cpu().numpy() - ref)) / np.max(np.abs(ref))) for x in xs)
    p.close()
    return err


# m = N - 1 chain positions against windows of 2, 8, 16 and 32
@pytest.mark.parametrize("n,nrhs", [(8, 1), (16, 8), (5, 8), (11, 1)])
@pytest.mark.parametrize("wd,later", [(1, 0), (3, 0), (4, 2), (5, 1)])
def test_window_edges_fp64(wd, later, n, nrhs):
    W = 1 << wd
    for m in sorted({0, 1, 2, W - 1, W, W + 1, W + 2, 2 * W - 1, 3 * W, 3 * W + 3}):
        assert _solve(3, m + 1, n, nrhs, "fp64", wd, later) <= 1e-11, m


@pytest.mark.parametrize("N,n,nrhs", [(1, 8, 1), (8, 16, 3), (9, 7, 8), (17, 16, 1), (40, 8, 2)])
def test_window_edges_fp32(N, n, nrhs):
    assert _solve(3, N, n, nrhs, "fp32", 0) <= 1e-10


@pytest.mark.parametrize("precision,tol", [("fp64", 1e-11), ("fp32", 1e-10)])
@pytest.mark.parametrize("n", [8, 6])
def test_two_waves_per_window(n, precision, tol):
    # 2 windows of 16 positions on each of 1200 chains: more waves than fit on the GPU
    assert _solve(1200, 20, n, 1, precision, 0) <= tol
