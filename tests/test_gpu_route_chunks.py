"""The data router's chunks, bf16: 16 tokens with the columns split over the waves, 64 tokens, two times 64; widths that leave waves or
parts of a step without columns, more patches than are folded at a time, two tiles of experts, ends of samples inside a chunk; and W_B too large
for the matrix-core kernel (split_d1032_n17).  KNOWN are sizes for which the chunk is looked up."""
import pytest

import test_gpu_parity as P
from test_route_chunks import chunk_tokens
from paper_2503_02495_amd import synth


def cfg(**kw):
    return P.small(d_h=32, n_m=4, d_e=32, k_m=2, c=1, k_a=1, dtype=synth.BF16, **kw)


pytestmark = pytest.mark.gpu

CONFIGS = {
    "split_d8": cfg(b=1, l=16, d=8, n_a=3, m=2),
    "split_d40_two_waves_idle": cfg(b=3, l=34, d=40, n_a=5, m=17),
    "split_d200": cfg(b=2, l=50, d=200, n_a=8, m=25),
    "split_d1032_n17": cfg(b=2, l=96, d=1032, n_a=17, m=6),
    "split_m130": cfg(b=2, l=260, d=96, n_a=3, m=130),
    "split_most_tokens": cfg(b=32, l=128, d=64, n_a=4, m=16),
    "one_token_more": cfg(b=17, l=241, d=64, n_a=4, m=1),
    "whole_d264_m65": cfg(b=64, l=65, d=264, n_a=8, m=65),
    "whole_d8": cfg(b=64, l=66, d=8, n_a=32, m=66),
    "twice_tail": cfg(b=97, l=510, d=40, n_a=6, m=51),
    "twice_n32_m64": cfg(b=48, l=1088, d=16, n_a=32, m=64),
}

# (config, tokens a chunk): on the matrix cores, W_B with 64 tokens' t1 and 8 KiB within 60 KiB
KNOWN = {
    "split_d520": (cfg(b=2, l=98, d=520, n_a=16, m=7), 16),              # 160 columns a wave, two register sets, 40 columns for the last wave
    "split_d776": (cfg(b=2, l=153, d=776, n_a=13, m=9), 16),             # 224 columns, 104 for the last wave
    "split_d1000": (cfg(b=3, l=95, d=1000, n_a=6, m=5), 16),             # 256 columns, 232 for the last wave
    "split_d640_n17": (cfg(b=2, l=102, d=640, n_a=17, m=6), 16),
    "split_d200_one_set": (cfg(b=2, l=50, d=200, n_a=8, m=5), 16),
    "whole_d264_m67": (cfg(b=33, l=134, d=264, n_a=8, m=67), 64),        # three sets, two groups of patches
    "whole_d72_n20": (cfg(b=33, l=130, d=72, n_a=20, m=10), 64),
    "twice_d264": (cfg(b=5, l=4020, d=264, n_a=8, m=60), 128),           # three sets of each 64 tokens, W_A fetched again between
    "twice_d392_n20": (cfg(b=5, l=4008, d=392, n_a=20, m=24), 128),
    "twice_d128": (cfg(b=5, l=4050, d=128, n_a=10, m=50), 128),
}


@pytest.mark.parametrize("name", list(KNOWN))
def test_route_parity_of_known_chunks(name, monkeypatch):
    c, tokens = KNOWN[name]
    np = (c.n_a + 15) // 16 * 16
    assert -(-c.d // 8) * (8 * np * 2 + (128 if np == 16 else 32)) + 64 * np * 4 + 8192 <= 60 * 1024
    assert chunk_tokens(c.b, c.l, c.d, c.n_a, c.m) == tokens
    monkeypatch.setitem(P.EDGE_CONFIGS, name, c)
    P.test_route_parity(name)


@pytest.mark.parametrize("name", list(CONFIGS))
def test_route_parity_chunks(name, monkeypatch):
    monkeypatch.setitem(P.EDGE_CONFIGS, name, CONFIGS[name])
    P.test_route_parity(name)
