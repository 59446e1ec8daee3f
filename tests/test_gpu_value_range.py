"""Values at the ends of what the storage types hold."""
import numpy as np
import pytest

import test_gpu_parity as P
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth

pytestmark = pytest.mark.gpu

R, GE, GP, CA = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT, B.FLAG_GATE_PATCH, B.FLAG_CAUSAL
BF = synth.BF16

RANGE = {
    "vr_dh8": P.small(b=2, l=35, d=40, n_a=3, d_h=8, m=5, c=2, k_a=2, n_m=3, d_e=8, k_m=2, dtype=BF),
    "vr_dh40": P.small(b=2, l=84, d=96, n_a=2, d_h=40, m=6, c=3, k_a=1, n_m=2, d_e=32, k_m=1, dtype=BF),
    "vr_dh96": P.small(b=2, l=84, d=64, n_a=2, d_h=96, m=6, c=3, k_a=1, n_m=2, d_e=32, k_m=1, dtype=BF),
    "vr_d72": P.small(b=2, l=192, d=72, n_a=3, d_h=64, m=6, c=4, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
}


@pytest.mark.parametrize("name", list(RANGE))
@pytest.mark.parametrize("power", [20, -24])
def test_smha_range_of_v(name, power, monkeypatch):
    """bf16 blocks off the 32-multiples: v and its probabilities are held in bf16 and fp32, so v may have any magnitude
    bf16 holds (2^20 here: past fp16's 65504; 2^-24: below its smallest value).  A power of two on W^v scales the exact
    result by itself: same bound as unscaled."""
    plain = synth.make_inputs

    def scaled(cfg, **kw):
        inp = plain(cfg, **kw)
        inp.wv = inp.wv * np.float32(2.0 ** power)
        return inp

    monkeypatch.setitem(P.EDGE_CONFIGS, name, RANGE[name])
    monkeypatch.setattr(synth, "make_inputs", scaled)
    print(f"range of v {name} 2^{power}", flush=True)
    P.run_smha_stage(name, 0)
    P.run_smha_variant(name, CA, 8, 0.2)
