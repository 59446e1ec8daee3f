"""Weight gradients whose experts are selected unequally: one by every sample, one by none, the others now and then, so that the parts of
the experts' lists differ in number and length.  Lists of whole pairs, of ranges of tokens (with a shorter last one), of picked patches;
more samples than a workgroup's table; as many experts as there may be; few or short parts and experts with many pairs, where all have
as many parts (skew), and lists cut into parts of equal length (equal).  Which of the two the library takes is its own rule's: EQUAL are sizes for
which it has been looked up that the parts are equal."""
import copy

import numpy as np
import pytest

import test_gpu_parity as P
import test_wgrad_lengths as lengths
import test_wgrad_parts as parts
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth

pytestmark = pytest.mark.gpu


def cfg(b, l, d, n, k, width, m=2, c=1, dtype=synth.BF16):
    return P.small(b=b, l=l, d=d, n_a=n, k_a=k, d_h=min(width, 64), m=m, c=c, n_m=n, k_m=k, d_e=width, dtype=dtype)


UOME = {
    "skew_ranges": cfg(3, 512, 64, 6, 2, 64),
    "skew_pairs": cfg(40, 32, 96, 8, 3, 160),
    "skew_n32": cfg(5, 192, 32, 32, 9, 32),
    "skew_many_pairs": cfg(100, 32, 64, 4, 2, 32),
    "skew_any_short_range": cfg(3, 397, 72, 5, 2, 56, m=1),
    "skew_f32": cfg(5, 260, 40, 7, 3, 136, dtype=synth.F32),
    "skew_f32_two_chunks": cfg(131, 20, 40, 9, 2, 24, dtype=synth.F32),
    "equal_by_sample": cfg(6, 2048, 32, 6, 2, 64),
    "equal_pairs": cfg(24, 512, 32, 4, 2, 32),
    "equal_any_short_range": cfg(4, 2500, 40, 5, 2, 24, m=1),
    "equal_f32": cfg(3, 4400, 40, 4, 2, 24, dtype=synth.F32),
    "equal_two_chunks": cfg(131, 162, 40, 9, 1, 24),
    "skew_any_many_pairs": cfg(150, 14, 40, 4, 2, 72),
}
SMHA = {
    "skew_sm": cfg(6, 256, 64, 5, 2, 64, m=8, c=3),
    "skew_sm_n32": cfg(4, 128, 32, 32, 9, 32, m=4, c=2),
    "skew_sm_long_lists": cfg(20, 512, 32, 6, 2, 32, m=16, c=9),
    "equal_sm": cfg(6, 512, 64, 5, 2, 64, m=16, c=8),
    "equal_sm_f32": cfg(5, 768, 40, 7, 3, 24, m=12, c=9, dtype=synth.F32),
    "equal_sm_two_chunks": cfg(131, 200, 40, 9, 1, 24, m=5, c=4),
    "skew_sm_f32": cfg(5, 77, 40, 7, 3, 24, m=7, c=4, dtype=synth.F32),
    "skew_sm_two_chunks": cfg(131, 14, 40, 9, 2, 24, m=2, c=2),
}

EQUAL_UOME = {   # with the average number of parts an expert off the 32-grid
    "n32_k9": (cfg(4, 2048, 32, 32, 9, 32), 0),
    "by_sample": (cfg(13, 1536, 64, 8, 2, 96), 0),
    "any_n32_k9": (cfg(4, 2500, 40, 32, 9, 24, m=1), 8),
    "any_short_last_range": (cfg(9, 1364, 72, 16, 5, 40, m=1), 8),
    "f32_n32_k10": (cfg(3, 3001, 40, 32, 10, 24, m=1, dtype=synth.F32), 8),
    "f32_few_pairs": (cfg(3, 4400, 40, 4, 2, 24, dtype=synth.F32), 8),
    "two_chunks": (cfg(131, 460, 40, 20, 2, 24), 4),
    "f32_two_chunks": (cfg(140, 470, 24, 21, 3, 40, dtype=synth.F32), 4),
}
EQUAL_SMHA = {   # with the most there can be
    "n32_k9": (cfg(4, 512, 32, 32, 9, 32, m=16, c=15), 0),
    "f32_n32_k9": (cfg(4, 528, 40, 32, 9, 24, m=16, c=15, dtype=synth.F32), 2),
    "two_chunks": (cfg(131, 640, 40, 20, 2, 24, m=8, c=7), 5),
    "f32_two_chunks": (cfg(131, 648, 40, 20, 2, 24, m=8, c=7, dtype=synth.F32), 5),
}


@pytest.fixture(autouse=True)
def _skewed(monkeypatch):
    plain = P.oracle.route

    def route(x, n, k, *args, **kw):
        out = copy.copy(plain(x, n, k, *args, **kw))
        rng = np.random.default_rng(n * 1000 + k)
        rows = [np.sort(np.append(rng.choice(np.arange(1, n - 1), k - 1, replace=False), 0)) for _ in range(x.shape[0])]
        ids = np.asarray(rows, out.expert_id.dtype)
        return out._replace(expert_id=ids) if hasattr(out, "_replace") else (setattr(out, "expert_id", ids), out)[1]

    monkeypatch.setattr(P.oracle, "route", route)


@pytest.mark.parametrize("name", list(UOME))
def test_uome_backward_of_skewed_selections(name, monkeypatch):
    monkeypatch.setitem(P.BWD_CONFIGS, name, UOME[name])
    P.test_uome_backward_parity(name, P.R | P.GE)


@pytest.mark.parametrize("name", list(SMHA))
def test_smha_backward_of_skewed_selections(name, monkeypatch):
    monkeypatch.setitem(P.SMHA_BWD_CONFIGS, name, SMHA[name])
    P.run_smha_backward(name, P.R | P.GE | P.GP, 0)


@pytest.fixture(scope="module")
def plans(tmp_path_factory):
    return lengths.build(tmp_path_factory.mktemp("plan"))


@pytest.mark.parametrize("name", list(EQUAL_UOME))
def test_uome_backward_in_equal_parts(name, plans, monkeypatch):
    c, s = EQUAL_UOME[name]
    if s:
        assert parts.uome_parts(c.b, c.l, c.d, c.n_m, c.k_m, c.d_e, B.F32 if c.dtype == synth.F32 else B.BF16) == s * -(-c.b // 128)
        plan = lengths.call(plans.any_plan, c.b, c.l, c.d, c.n_m, c.k_m, s, c.dtype == synth.F32)
    else:
        plan = lengths.call(plans.grid_plan, c.b, c.l, c.d, c.n_m, c.k_m, c.d_e)
    assert plan["each"] == 0
    monkeypatch.setitem(P.BWD_CONFIGS, name, c)
    P.test_uome_backward_parity(name, P.R | P.GE)


@pytest.mark.parametrize("name", list(EQUAL_SMHA))
def test_smha_backward_in_equal_parts(name, plans, monkeypatch):
    c, s = EQUAL_SMHA[name]
    l_p = c.l // c.m
    some = [lengths.call(plans.any_patch_plan, c.b, c.n_a, c.k_a, c.c, l_p, t) for t in range(2, s + 1)] if s else \
           [lengths.call(plans.patch_plan, c.b, c.n_a, c.k_a, c.c, l_p, 4, c.d_h, c.d)]
    assert all(plan["each"] == 0 for plan in some)
    monkeypatch.setitem(P.SMHA_BWD_CONFIGS, name, c)
    P.run_smha_backward(name, P.R | P.GE | P.GP, 0)
