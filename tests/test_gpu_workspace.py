"""Plan workspaces: the buffers of the forward substitution inside the factorization exist only
where it takes place (n <= 32, up to eight right-hand sides), for as many right-hand sides."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("precision,size", [("fp64", 8), ("fp32", 4)])
@pytest.mark.parametrize("n,below", [(8, 8), (16, 8), (32, 8), (40, 1), (64, 4)])
def test_no_fused_buffers_beyond_the_fused_right_hand_sides(n, below, precision, size):
    from paper_2609_29977_amd import bmpc
    S, N, passes = 16, 200, {}

    def bytes_of(nrhs):
        p = bmpc.Plan(S, N, n, nrhs, precision)
        c = p.cost()
        p.close()
        return c.workspace_bytes

    # what one more right-hand side needs: y, w, x_0 and the residual, its norms and their
    # partial maxima (2 x 1024), per residual workgroup (at least 8 stages each) a maximum;
    # 256-byte allocations.  x_1's and the windows' vectors of a pass would come on top
    one = S * N * n * size + S * n * 8 + n * 8 + (S * N + 1) * n * 8
    one += (2 + 2 * 1024 + S * (N + 7) // 8) * 8 + 32 * 256
    for extra in (1, 8):
        assert bytes_of(below + extra) - bytes_of(below) <= extra * one
