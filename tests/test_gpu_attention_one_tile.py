"""fp32 attention backward at the line between a tile a wave and several: 32, 64 and 128 rows with one, two and four waves per
block, one row less (a partly empty last tile) and one more (a wave with two tiles, the others with one), for each padded
width, and launches of more than 1024 blocks on either side (one wave with all tiles of longer units, for each padded width).  Same oracle and bounds as the other backward tests."""
import pytest

import test_gpu_parity as P
from paper_2503_02495_amd import synth

pytestmark = pytest.mark.gpu

R, GE, GP, CA = P.R, P.GE, P.GP, P.CA
BF = synth.BF16


def shape(b, rows, d_h, n=2, **kw):
    return P.small(b=b, l=rows, d=40, n_a=n, d_h=d_h, m=1, c=1, k_a=n, n_m=2, d_e=32, k_m=1, **kw)


CONFIGS = {f"one_{rows}_dh{d_h}": shape(2, rows, d_h, dtype=BF if rows % 2 else synth.F32)
           for rows in (31, 32, 33, 64, 65, 127, 128, 129) for d_h in (24, 64, 128)}
CONFIGS["one_520_units"] = shape(130, 60, 64, n=4)
CONFIGS["several_206_units"] = shape(103, 130, 24)
CONFIGS["several_206_units_dh64"] = shape(103, 130, 64)
CONFIGS["several_206_units_dh128"] = shape(103, 130, 128, dtype=BF)


@pytest.mark.parametrize("name", list(CONFIGS))
@pytest.mark.parametrize("flags,pad_frac", [(0, 0.0), (CA | R | GE | GP, 0.2)])
def test_smha_backward_one_tile(name, flags, pad_frac, monkeypatch):
    print(name, flags, flush=True)
    monkeypatch.setitem(P.SMHA_BWD_CONFIGS, name, CONFIGS[name])
    P.run_smha_backward(name, flags, 0, pad_frac=pad_frac)
