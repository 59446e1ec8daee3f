"""fp32 routers below 8192 tokens in chunks of 4 to 12 tokens: the smallest chunks and the largest, a last one that is shorter, samples shorter
than a chunk, the longest lists of chunks that the selection adds up itself (16384 partial logits a sample) and one past it, more logits than
it takes."""
import pytest

import test_gpu_parity as P

pytestmark = pytest.mark.gpu

CONFIGS = {
    "short_chunks_of_4": P.small(b=3, l=42, d=40, n_a=3, d_h=8, m=6, c=2, k_a=2, n_m=3, d_e=8, k_m=1),
    "short_sample_of_2": P.small(b=5, l=2, d=24, n_a=2, d_h=8, m=2, c=1, k_a=1, n_m=2, d_e=8, k_m=1),
    "short_chunks_of_12": P.small(b=13, l=500, d=16, n_a=4, d_h=8, m=10, c=3, k_a=2, n_m=4, d_e=8, k_m=2, router_noise=True),
    "short_logits_16384": P.small(b=1, l=512, d=16, n_a=8, d_h=8, m=16, c=4, k_a=2, n_m=8, d_e=8, k_m=2),
    "short_logits_past_16384": P.small(b=1, l=528, d=16, n_a=8, d_h=8, m=16, c=4, k_a=2, n_m=8, d_e=8, k_m=2),
    "short_logits_544": P.small(b=2, l=136, d=16, n_a=8, d_h=8, m=68, c=9, k_a=2, n_m=4, d_e=8, k_m=2),
}


@pytest.mark.parametrize("name", list(CONFIGS))
def test_route_parity_short_chunks(name, monkeypatch):
    monkeypatch.setitem(P.EDGE_CONFIGS, name, CONFIGS[name])
    P.test_route_parity(name)
