"""Every factor pass that a plan may run fits the 160 KB of LDS of a compute unit, the last
one included, which holds x_1 and C on top of its window at n <= 16.

Host: the LDS of each pass of the planned depths, from the layouts of the pass kernels
(n <= 16: a window's 2 W - 1 blocks, two more in the last pass, and W + 1 vectors; 17..32: 2 Tw +
3 blocks and Tw + 3 vectors; rows of NMAX + 1 entries, 34 at NMAX = 32), over precision, block
size, fused right-hand sides, depths and chain lengths.  GPU: the shapes whose last pass
decides the depth, against the FP64 oracle with the parity suite's tolerances (1e-11 FP64,
1e-10 FP32 with refinement)."""
import numpy as np
import pytest

from paper_2609_29977_amd import bmpc

BUDGET = 160 * 1024


def _pass_bytes(n, size, Tw, mk, nrhs):
    final = mk < (1 << Tw)
    if n <= 16:
        nmax = 8 if n <= 8 else 16
        Tw = min(Tw, mk.bit_length()) if final and mk else Tw
        W = min(1 << Tw, mk + 1) if mk else 2
        return ((2 * W - 1 + 2 * final) * nmax * (nmax + 1) + (W + 1) * nrhs * nmax) * size
    return ((2 * Tw + 3) * 32 * 34 + (Tw + 3) * nrhs * 32) * size


@pytest.mark.parametrize("precision,size", [("fp64", 8), ("fp32", 4)])
@pytest.mark.parametrize("n", [3, 8, 9, 16, 17, 32])
@pytest.mark.parametrize("depth", [1, 2, 3, 4, 5, 6])
def test_every_planned_pass_fits(depth, n, precision, size):
    for nrhs in range(1, 10):
        for N in [1, 2] + [k + d for k in (4, 8, 16, 32, 64, 128, 256, 4096) for d in (-1, 0, 1)]:
            for later in (0, depth, 6):
                c = bmpc.cost_model(2, N, n, nrhs, precision, window_depth=depth,
                                    later_depth=later)
                mk, Tw, passes = N - 1, c.window_depth, 0
                while True:
                    need = _pass_bytes(n, size, Tw, mk, min(nrhs, 8))
                    assert need <= BUDGET, (nrhs, N, later, passes, Tw, mk, need)
                    passes += 1
                    if mk < (1 << Tw):
                        break
                    mk, Tw = mk >> Tw, c.later_depth
                assert passes == c.passes


# six right-hand sides: a window of 32 (FP64) or 64 (FP32) positions fits, the last pass over
# 31 or 63 of them does not
@pytest.mark.gpu
@pytest.mark.parametrize("precision,N,depth,tol", [("fp64", 32, 5, 1e-11), ("fp32", 64, 6, 1e-10)])
def test_last_pass_over_a_full_window(precision, N, depth, tol):
    import torch

    from oracle import oracle
    from synth.branch_system import make_system
    s = make_system(3, N, 16, 6, 1e-2, 11)
    ref, info = oracle.solve(s.D, s.E, s.C, s.R, s.b, nthreads=8)
    assert info == 0
    D, E, C, R, b = (torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")
                     for a in (s.D, s.E, s.C, s.R, s.b))
    p = bmpc.Plan(3, N, 16, 6, precision, depth)
    x = (p.factor_solve(D, E, C, R, b) if precision == "fp64"
         else p.factor_refine(D, E, C, R, b, tol=1e-13, max_iters=10))
    assert p.info() == 0
    assert float(np.max(np.abs(x.cpu().numpy() - ref)) / np.max(np.abs(ref))) <= tol
    p.close()
