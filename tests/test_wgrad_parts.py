"""How many parts the any-shape weight gradients are cut into, read off the workspace sizes (no GPU)."""
import pytest

from paper_2503_02495_amd import binding as B


def uome_parts(b, l, d, n, k, d_e, dtype):
    nbytes = B.uome_backward_workspace_bytes(B.block_desc(b, l, d, n, k, 1, 1, d_e, dtype, 0))
    return (nbytes - 2 * b * l * k * d_e * 4) // (2 * n * d * d_e * 4)


@pytest.mark.parametrize("n,want", [(6, 7), (8, 8), (12, 7), (16, 4)])
def test_workgroups_spread_evenly_over_the_compute_units(n, want):
    """128 samples of 196 tokens, d 384, d_e 256 in bf16: 12 n workgroups a part on 256 units.  6 experts: eight parts
    are 576, three on some units, seven 504, two; 8 experts: eight are 768, three on every unit, and fewer only lengthen the longest sum; 16
    (at most five parts): four are 768 again."""
    assert uome_parts(128, 196, 384, n, n // 2, 256, B.BF16) == want


def test_parts_follow_the_tiles_of_fp32():
    """24 samples of 500 tokens, d 768, d_e 192: in fp32 five parts are 1200 tiles of 64x64 or 360 of 64x128, not 240 of 128x128."""
    assert uome_parts(24, 500, 768, 4, 2, 192, B.F32) >= 6
    assert uome_parts(8, 77, 200, 4, 2, 136, B.F32) == 8
