"""The data router's chunks, bf16: 16 tokens with the columns split over the waves, 64 tokens, two times 64; widths that leave waves or
parts of a step without columns, more patches than are folded at a time, two tiles of experts, ends of samples inside a chunk."""
import pytest

import test_gpu_parity as P
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


@pytest.mark.parametrize("name", list(CONFIGS))
def test_route_parity_chunks(name, monkeypatch):
    monkeypatch.setitem(P.EDGE_CONFIGS, name, CONFIGS[name])
    P.test_route_parity(name)
