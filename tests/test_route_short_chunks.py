"""How many tokens a workgroup of the fp32 routers takes, read off the workspace sizes (no GPU)."""
import pytest

from paper_2503_02495_amd import binding as B


def up(nbytes):
    return -(-nbytes // 256) * 256


def chunk_tokens(b, l, d, n, m):
    """(expert router's, data router's) of 4, 8, 12, 16 and more, by the partial sums of a block whose other buffers are known."""
    got = B.workspace_bytes(None, B.block_desc(b, l, d, n, 1, m, 1, 8, B.F32, 0))
    c = 1
    rest = up(b * l * 8 * 4) + up(b * 4) + up(b * n * 4) + up(b * n * c * 4) + up(b * n * m * 4) + up(b * n * m * 4)   # hidden, routing, summed logits
    fits = {(t, td) for t in (4, 8, 12, 16) for td in (4, 8, 12, 16) if td >= t and rest + up(-(-l // t) * b * n * 4) + up(-(-l // td) * b * n * m * 4) == got}
    assert len(fits) == 1, (got - rest, fits)
    return fits.pop()


@pytest.mark.parametrize("b,l,d,n,m,want", [
    (2, 64, 64, 4, 8, (4, 4)), (8, 512, 512, 8, 16, (8, 8)), (1, 240, 608, 20, 6, (4, 4)),   # workgroups for idle compute units
    (28, 217, 184, 14, 7, (16, 16)),                     # shorter ones: more chunks on the fullest XCD than they are shorter by
    (15, 504, 1032, 8, 14, (16, 16)),                    # W_B leaves room for four workgroups a compute unit
    (1, 2006, 784, 12, 34, (16, 16)), (1, 1632, 992, 11, 51, (16, 16)),   # a large W_E is read in longer runs
    (6, 442, 488, 14, 34, (16, 16)),                     # 476 logits: the data router keeps its 16 tokens, and the launch is as long as they take
    (2, 2816, 232, 23, 256, (16, 16)),                   # 30 KB more for shorter chunks would not fit the fixed scratch of uoe_route_static
    (33, 162, 56, 32, 3, (8, 8)), (20, 406, 104, 24, 14, (16, 16)),       # whole rounds of workgroups with more than 16 experts
])
def test_tokens_of_a_chunk(b, l, d, n, m, want):
    assert chunk_tokens(b, l, d, n, m) == want
