"""QP assembly (bmpc_assemble_qp): D and R are exactly symmetric for a symmetric Q; row counts that
leave a step of four rows incomplete, and zero entries, with a delta whose reciprocal is
infinite.  Reference: the link sums in numpy FP64, with the bound of the assembly's other
tests (1e-13 of the largest entry)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).to("cuda")


def _assemble(*args):
    from paper_2609_29977_amd import bmpc
    return [x.cpu().numpy() for x in bmpc.assemble_qp(*[_dev(a) for a in args[:4]], *args[4:])]


@pytest.mark.parametrize("n,mi", [(5, 1), (16, 7), (32, 30)])
def test_denormal_delta(n, mi):
    rng = np.random.default_rng(n)
    S, N, n2 = 2, 5, 2 * n
    Q = rng.standard_normal((S, N + 1, n2, n2))
    G = rng.standard_normal((S, N + 1, mi, n2))
    w = rng.uniform(0.5, 2.0, (S, N + 1, mi))
    M = Q + np.swapaxes(G, 2, 3) @ (G / w[..., None])
    D, E, C, R = _assemble(Q, np.zeros((S, N + 1, 0, n2)), G, w, 0.0, 1e-310)
    for got, ref in ((D, M[:, :N, n:, n:] + M[:, 1:, :n, :n]), (E, M[:, 1:N, n:, :n]),
                     (C, M[:, 0, :n, n:]), (R, M[:, 0, :n, :n].sum(0))):
        assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(M))


@pytest.mark.parametrize("S,N,n,me,mi", [(1, 1, 1, 1, 1), (3, 9, 7, 3, 5), (2, 17, 16, 12, 32),
                                         (5, 8, 17, 4, 7), (2, 10, 32, 64, 128)])
def test_symmetric_for_a_symmetric_cost(S, N, n, me, mi):
    rng = np.random.default_rng(n + N)
    n2 = 2 * n
    Q = rng.standard_normal((S, N + 1, n2, n2))
    Q = Q + np.swapaxes(Q, 2, 3)
    A = rng.standard_normal((S, N + 1, me, n2))
    G = rng.standard_normal((S, N + 1, mi, n2))
    w = 10.0 ** rng.uniform(-3, 1, (S, N + 1, mi))
    D, _, _, R = _assemble(Q, A, G, w, 1e-3, 1e-2)
    assert np.array_equal(D, np.swapaxes(D, -1, -2)) and np.array_equal(R, R.T)


def test_denormal_delta_with_zero_entries():
    rng = np.random.default_rng(3)
    S, N, n, me, delta = 2, 4, 6, 4, 1e-310
    A = 1e-10 * rng.standard_normal((S, N + 1, me, 2 * n)) * (rng.random((S, N + 1, me, 2 * n)) < 0.5)
    Q = np.zeros((S, N + 1, 2 * n, 2 * n))
    X = A / np.sqrt(delta)
    M = np.swapaxes(X, 2, 3) @ X
    D, E, C, R = _assemble(Q, A, np.zeros((S, N + 1, 0, 2 * n)), np.zeros((S, N + 1, 0)), 0.0, delta)
    for got, ref in ((D, M[:, :N, n:, n:] + M[:, 1:, :n, :n]), (E, M[:, 1:N, n:, :n]),
                     (C, M[:, 0, :n, n:]), (R, M[:, 0, :n, :n].sum(0))):
        assert np.max(np.abs(got - ref)) <= 1e-13 * np.max(np.abs(M))
