"""Depth of the factor passes after the first, from the cost model (host): four levels for blocks of
9..16 where that ends the chain with the second pass, up to 512 scenarios or with eight
positions left; the same for a batch of any number of such systems."""
import pytest

from paper_2609_29977_amd import bmpc


@pytest.mark.parametrize("precision", ["fp64", "fp32"])
@pytest.mark.parametrize("n", [9, 16])
@pytest.mark.parametrize("S,N,later", [(4, 64, 3), (4, 65, 4), (512, 100, 4), (513, 100, 3),
                                       (513, 72, 4), (513, 73, 3), (512, 128, 4), (4096, 128, 3),
                                       (512, 129, 3), (4096, 65, 4)])
def test_later_depth(S, N, later, n, precision):
    for systems in (1, 7):
        c = bmpc.cost_model(S, N, n, 1, precision, num_systems=systems)
        assert (c.window_depth, c.later_depth) == (3, later)


@pytest.mark.parametrize("n,depth", [(8, 4), (17, 3), (32, 3), (33, 1)])
def test_other_block_sizes_keep_the_first_depth(n, depth):
    for S in (4, 1024):
        c = bmpc.cost_model(S, 100, n, 1, "fp64")
        assert (c.window_depth, c.later_depth) == (depth, depth)
