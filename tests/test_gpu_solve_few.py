"""Solves of few right-hand sides with the kernels that hold a block in the registers of four
waves: block sizes at the edges of their classes (full and padded), chains of 0 to 8
levels, the launch flags, a last chunk of few right-hand sides behind sixteen; the root
step either side of its scenario counts.  Reference: the FP64 oracle with the parity
suite's tolerances (1e-11 FP64, 1e-10 FP32 with refinement)."""
import numpy as np
import pytest

from oracle import oracle
from synth.branch_system import make_system

pytestmark = pytest.mark.gpu


def _dev(a):
    import torch
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda:0")


def _check(S, N, n, nrhs, precision, flags=0):
    from paper_2609_29977_amd import bmpc
    s = make_system(S, N, n, nrhs, 1e-2, 90 + N + n)
    ref, info = oracle.solve(s.D, s.E, s.C, s.R, s.b, nthreads=8)
    assert info == 0
    K = (_dev(s.D), _dev(s.E) if N > 1 else None, _dev(s.C), _dev(s.R))
    b = _dev(s.b)
    p = bmpc.Plan(S, N, n, nrhs, precision, flags=flags)
    p.factor(*K)
    x = p.solve(b) if precision == "fp64" else p.refine(*K, b, tol=1e-13, max_iters=10)
    assert p.info() == 0
    err = float(np.max(np.abs(x.cpu().numpy() - ref)) / np.max(np.abs(ref)))
    assert err <= (1e-11 if precision == "fp64" else 1e-10), (N, err)
    p.close()


# either side of the chains whose top levels share a launch (512, 256 above n = 16), and of the
# scenarios that the root step reads in one go (128, 512)
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("S", [127, 129, 255, 257, 511, 514])
@pytest.mark.parametrize("n,nrhs", [(8, 2), (8, 3), (16, 1), (12, 5), (21, 2), (32, 3), (32, 6)])
def test_chain_counts(n, nrhs, S, precision):
    _check(S, 12, n, nrhs, precision)


SIZES64 = [(49, 1), (49, 4), (50, 3), (63, 2), (64, 1), (64, 4), (64, 5), (57, 18)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", SIZES64)
def test_blocks_over_48(n, nrhs, precision):
    for N in (1, 2, 7, 40, 130):
        _check(3, N, n, nrhs, precision)
    for flags in (1, 2, 3):
        _check(2, 21, n, nrhs, precision, flags)
