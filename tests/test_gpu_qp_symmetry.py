"""QP assembly (bmpc_assemble_qp): row counts that leave a step of four rows incomplete with a delta
whose reciprocal is infinite.  Reference: the link sums in numpy FP64, with the bound of
the assembly's other tests (1e-13 of the largest entry)."""
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
