"""Room for the routers of a UoME block that selects experts only (c = m): uoe_layer_forward routes it with one patch, whatever m its description has, so
the workspace has to hold either plan of the routers' chunks (read off the workspace sizes, no GPU)."""
import random

import pytest

from paper_2503_02495_amd import binding as B


def block_bytes(b, l, d, n, m, dtype):
    return B.workspace_bytes(None, B.block_desc(b, l, d, n, 1, m, m, 8, dtype, 0))


@pytest.mark.parametrize("b,l,d,n,m,dtype", [(1, 4096, 192, 16, 2, B.BF16), (1, 3672, 288, 29, 2, B.BF16), (1, 3015, 344, 19, 3, B.BF16),
                                             (1, 2618, 64, 25, 2, B.F32), (1, 2247, 272, 28, 3, B.F32)])
def test_one_patch_fits(b, l, d, n, m, dtype):
    assert block_bytes(b, l, d, n, m, dtype) >= block_bytes(b, l, d, n, 1, dtype)


def test_one_patch_fits_over_the_sizes():
    rng = random.Random(1)
    for _ in range(20000):
        dtype, n, m, b = rng.choice((B.F32, B.BF16)), rng.randint(1, 32), rng.choice((2, 3, 4, 5, 7, 8, 16)), rng.choice((1, 2, 3, 8, 33, 64))
        l, d = m * rng.randint(1, 4096 // m), 8 * rng.randint(1, 128)
        assert block_bytes(b, l, d, n, m, dtype) >= block_bytes(b, l, d, n, 1, dtype), (b, l, d, n, m, dtype)
