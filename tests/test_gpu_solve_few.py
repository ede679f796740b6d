"""Solves of few right-hand sides with the kernels that hold a block in the registers of one or
four waves: block sizes at the edges of their classes (full and padded), chains of 0 to 9
levels, the launch flags, a last chunk of few right-hand sides behind sixteen, more
scenarios than a grid dimension holds; and of any number either side of the chains whose
top levels share a launch.  Reference: the FP64 oracle with the parity suite's tolerances
(1e-11 FP64, 1e-10 FP32 with refinement); merged launches, ragged plans and batches are
bitwise the level launches and the systems' own plans."""
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


SIZES = [(1, 1), (1, 3), (1, 6), (2, 17), (5, 2), (8, 1), (8, 2), (8, 3), (9, 2), (12, 1), (15, 2),
         (16, 1), (16, 2), (17, 1), (17, 2), (24, 2), (31, 1), (31, 2), (32, 1), (32, 2), (32, 3),
         (13, 17), (32, 18)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", SIZES)
def test_blocks_up_to_32(n, nrhs, precision):
    for N in (1, 2, 3, 5, 21, 140, 258):  # 0 to 9 levels; x_1 with up to 4 and more pulls
        _check(2, N, n, nrhs, precision)
    for flags in (1, 2, 3):
        _check(2, 40, n, nrhs, precision, flags)


# either side of the chains whose top levels share a launch (512, 256 above n = 16), of the
# scenarios that the root step reads in one go (128, 512) and of those that decide which
# kernels take two or three right-hand sides (32, 256)
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("S", [32, 33, 127, 129, 255, 257, 511, 514])
@pytest.mark.parametrize("n,nrhs", [(8, 2), (8, 3), (16, 1), (12, 5), (12, 3), (21, 2), (19, 3),
                                    (24, 2), (28, 2), (32, 3), (32, 6)])
def test_chain_counts(n, nrhs, S, precision):
    for N in (12, 6, 36):
        _check(S, N, n, nrhs, precision)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(4, 1), (4, 2), (3, 3)])
def test_more_scenarios_than_a_grid_dimension(n, nrhs, precision):
    _check(66000, 4, n, nrhs, precision)


# the sums do not depend on which levels share a launch
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(8, 2), (8, 3), (13, 1), (13, 2), (16, 2), (16, 4), (20, 1),
                                    (24, 2), (31, 6), (32, 3), (32, 9), (40, 1), (48, 16),
                                    (64, 2), (64, 7)])
def test_merged_top_levels_are_bitwise_the_level_launches(n, nrhs, precision):
    from paper_2609_29977_amd import bmpc
    S, N = 3, 45
    s = make_system(S, N, n, nrhs, 1e-2, 7)
    K = tuple(_dev(a) for a in (s.D, s.E, s.C, s.R))
    b = _dev(s.b)
    outs = []
    for flags in (0, bmpc.FLAG_NO_BWD_TOP_MERGE):
        p = bmpc.Plan(S, N, n, nrhs, precision, flags=flags)
        p.factor(*K)
        outs.append(p.solve(b).cpu().numpy())
        p.close()
    assert np.array_equal(*outs)


# 640 chains in the batch, 40 in each of its systems' own plans: single and merged top levels
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("nrhs", [1, 2, 3, 4])
def test_ragged_beyond_the_merged_launches_is_bitwise_its_plans(nrhs, precision):
    import torch

    from paper_2609_29977_amd import bmpc
    shapes = [(40, N, n) for N, n in ((9, 8), (20, 8), (33, 5), (12, 12), (40, 16), (7, 15),
                                      (21, 20), (16, 32), (35, 24), (10, 31), (3, 9), (5, 16),
                                      (1, 8), (2, 32), (18, 27), (24, 11))]
    systems = [make_system(S, N, n, nrhs, 1e-2, 170 + i) for i, (S, N, n) in enumerate(shapes)]
    rp = bmpc.RaggedPlan([(S, N, n, nrhs) for S, N, n in shapes], precision)
    parts = lambda name: [_dev(getattr(s, name)) for s in systems]
    rp.factor(rp.pack(0, parts("D")), rp.pack(1, [_dev(s.E) if s.N > 1 else None for s in systems]),
              rp.pack(2, parts("C")), rp.pack(3, parts("R")))
    x = rp.solve(rp.pack(4, parts("b")))
    for i, s in enumerate(systems):
        p = bmpc.Plan(s.S, s.N, s.n, nrhs, precision)
        p.factor(_dev(s.D), _dev(s.E) if s.N > 1 else None, _dev(s.C), _dev(s.R))
        assert torch.equal(rp.unpack(4, x, i), p.solve(_dev(s.b)).reshape(-1)), shapes[i]
        p.close()
    rp.close()


# a batch beyond them and beyond a grid dimension
@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("B,S,N,n,nrhs", [(20, 40, 21, 16, 2), (20, 40, 21, 24, 1),
                                          (6, 60, 10, 48, 1), (66000, 1, 3, 4, 2)])
def test_batch_is_bitwise_its_plans(B, S, N, n, nrhs, precision):
    import torch

    from paper_2609_29977_amd import bmpc
    one = make_system(S, N, n, nrhs, 1e-2, 5)
    K = [_dev(a) for a in (one.D, one.E, one.C, one.R)]
    p = bmpc.Plan(S, N, n, nrhs, precision)
    p.factor(*K)
    b = _dev(one.b)
    own = [p.solve(b), p.solve(2 * b)]
    p.close()
    p = bmpc.Plan(S, N, n, nrhs, precision, num_systems=B)
    p.factor(*[t.unsqueeze(0).expand(B, *t.shape).contiguous() for t in K])
    bb = b.unsqueeze(0).expand(B, *b.shape).contiguous()
    bb[1::2] *= 2
    x = p.solve(bb).view(B, *b.shape)
    p.close()
    for i in (0, 1, B // 2, B - 2, B - 1):
        assert torch.equal(x[i], own[i % 2]), i
    assert torch.equal(x[0::2].amax(0), own[0]) and torch.equal(x[0::2].amin(0), own[0])


SIZES64 = [(49, 1), (49, 4), (50, 3), (63, 2), (64, 1), (64, 4), (64, 5), (57, 18)]


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", SIZES64)
def test_blocks_over_48(n, nrhs, precision):
    for N in (1, 2, 7, 40, 130):
        _check(3, N, n, nrhs, precision)
    for flags in (1, 2, 3):
        _check(2, 21, n, nrhs, precision, flags)


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n,nrhs", [(33, 1), (40, 2), (47, 1), (48, 2), (48, 3)])
def test_short_chains_of_blocks_over_32(n, nrhs, precision):
    for S, N in ((1, 1), (3, 2), (512, 2), (513, 2), (3, 3)):
        _check(S, N, n, nrhs, precision)
