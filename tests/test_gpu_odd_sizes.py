"""GPU parity of the kernels that take widths and token counts no tile divides, and of the fp32 matrix
path, at the sizes where they can go wrong: one element past and one short of a tile, K segments that end
inside a K-step, heads one step below and above a padded width, and both tile choices.  Same oracle,
metric and bounds as test_gpu_parity (1e-4 in fp32, 2e-2 in bf16)."""
import math

import pytest

import test_gpu_parity as P
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth

pytestmark = pytest.mark.gpu

R, GE, GP, CA = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT, B.FLAG_GATE_PATCH, B.FLAG_CAUSAL
BF = synth.BF16
ODD = {
    # bf16: head widths around the padded 32 / 64 / 128, K ending 8, 16 or 24 into a K-step
    "odd_dh8": P.small(b=2, l=35, d=40, n_a=3, d_h=8, m=5, c=2, k_a=2, n_m=3, d_e=8, k_m=2, dtype=BF),
    "odd_dh40": P.small(b=3, l=105, d=72, n_a=4, d_h=40, m=15, c=4, k_a=3, n_m=4, d_e=56, k_m=2, dtype=BF),
    "odd_dh72": P.small(b=2, l=198, d=104, n_a=3, d_h=72, m=6, c=2, k_a=2, n_m=2, d_e=88, k_m=1, dtype=BF),
    "odd_dh120": P.small(b=2, l=130, d=136, n_a=2, d_h=120, m=2, c=1, k_a=1, n_m=2, d_e=136, k_m=2, dtype=BF),
    # units of 4096 keys (the last whose padding flags fit LDS), one patch more, and a last key tile of 8
    "flags_4096": P.small(b=1, l=8192, d=64, n_a=2, d_h=64, m=64, c=32, k_a=1, n_m=2, d_e=64, k_m=1, dtype=BF),
    "flags_4224": P.small(b=1, l=8192, d=64, n_a=2, d_h=64, m=64, c=33, k_a=1, n_m=2, d_e=64, k_m=1, dtype=BF),
    "flags_tail": P.small(b=2, l=272, d=64, n_a=2, d_h=128, m=2, c=1, k_a=1, n_m=2, d_e=64, k_m=1, dtype=BF),
    # enough 128-row tiles for the large-tile choice, rows and columns 8 past two tiles
    "odd_big": P.small(b=32, l=264, d=136, n_a=2, d_h=16, m=8, c=8, k_a=2, n_m=2, d_e=136, k_m=2, dtype=BF),
    # fp32: the same sizes (64x64 tiles there; every fp32 tile: test_gpu_f32_split.py), and the launch shapes of the fp32 attention: one or two
    # query blocks, one, two or four key splits
    "f32_big": P.small(b=32, l=264, d=136, n_a=2, d_h=16, m=8, c=8, k_a=2, n_m=2, d_e=136, k_m=2),
    "f32_many_units": P.small(b=64, l=264, d=40, n_a=2, d_h=40, m=8, c=8, k_a=2, n_m=2, d_e=24, k_m=1),
    "f32_one_tile": P.small(b=2, l=32, d=64, n_a=2, d_h=64, m=1, c=1, k_a=1, n_m=2, d_e=64, k_m=1),
    "f32_dh128": P.small(b=1, l=66, d=128, n_a=2, d_h=128, m=2, c=2, k_a=1, n_m=2, d_e=128, k_m=1),
}
P.EDGE_CONFIGS.update(ODD)
ODD_DS = {
    "odd_ds": P.small(b=3, l=140, d=72, n_a=3, d_h=40, m=10, c=3, k_a=2, n_m=4, d_e=56, k_m=3, m_m=10, c_m=4, dtype=BF),
    "f32_ds": P.small(b=2, l=330, d=40, n_a=2, d_h=8, m=5, c=2, k_a=1, n_m=3, d_e=136, k_m=2, m_m=5, c_m=3),
}
P.DS_CONFIGS.update(ODD_DS)


@pytest.fixture(autouse=True)
def _std(monkeypatch):
    """Weights of std 0.06: attention logits of std 0.06^2 d, 0.14 at d = 40 and 0.5 at d = 136, a nearly uniform softmax
    (test_smha_f32_logits_of_order_one has the other kind)."""
    monkeypatch.setattr(P, "w_std_for", lambda name: 0.06)


def order_one_logits(monkeypatch):
    """Weights of std sqrt(1.5 / d): attention logits of std 1.5, running maxima that move and key splits that differ."""
    plain = synth.make_inputs
    monkeypatch.setattr(synth, "make_inputs", lambda cfg, **kw: plain(cfg, w_std=math.sqrt(1.5 / cfg.d)))


@pytest.mark.parametrize("name", list(ODD))
@pytest.mark.parametrize("flags,rope_dim,pad_frac", [(0, 0, 0.0), (CA | R | GE | GP, 8, 0.3)])
def test_smha_odd_sizes(name, flags, rope_dim, pad_frac):
    print(f"smha odd {name} flags={flags}", flush=True)
    P.run_smha_variant(name, flags, rope_dim, pad_frac)


@pytest.mark.parametrize("name", [n for n in ODD if n.startswith("f32")])
@pytest.mark.parametrize("flags,pad_frac", [(0, 0.0), (CA | R | GE | GP, 0.3)])
def test_smha_f32_logits_of_order_one(name, flags, pad_frac, monkeypatch):
    order_one_logits(monkeypatch)
    print(f"smha logits of order one {name} flags={flags}", flush=True)
    P.run_smha_variant(name, flags, 0, pad_frac)


@pytest.mark.parametrize("name", list(ODD))
@pytest.mark.parametrize("flags", [0, R | GE])
def test_uome_odd_sizes(name, flags):
    print(f"uome odd {name} flags={flags}", flush=True)
    P.run_uome_stage(name, flags)


@pytest.mark.parametrize("name", list(ODD_DS))
@pytest.mark.parametrize("flags", [0, R | GE | GP])
def test_uome_data_selection_odd_sizes(name, flags):
    print(f"uome data selection odd {name} flags={flags}", flush=True)
    P.test_uome_data_selection_stage_parity(name, flags)


# --------------------------------------------------------------------------- backward passes
UOME_BWD = {
    "ub_odd": P.small(b=3, l=77, d=72, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=5, d_e=40, k_m=2, dtype=BF),
    # two chunks of samples in the weight gradients' segment tables
    "ub_b130": P.small(b=130, l=9, d=16, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=3, d_e=8, k_m=2, dtype=BF),
    "ub_f32_b130": P.small(b=130, l=9, d=16, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=3, d_e=8, k_m=2),
    # rows of (hi, lo) pairs that are rewritten in place (2048) and the first length that is not
    "ub_in_place": P.small(b=2, l=20, d=16, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=2, d_e=2048, k_m=1, dtype=BF),
    "ub_wide": P.small(b=2, l=20, d=16, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=2, d_e=2056, k_m=1, dtype=BF),
    # ranges of the token axis, the last one short; one expert, one sample
    "ub_ranges": P.small(b=1, l=1100, d=40, n_a=1, d_h=8, m=1, c=1, k_a=1, n_m=1, d_e=24, k_m=1, dtype=BF),
    # fp32: 128x128 tiles in the launch of Z and dH; weight gradients with five of the eight token ranges empty, the last one of 13
    # tokens inside a K-step; d_u of one short K-step
    "ub_f32_big": P.small(b=32, l=264, d=136, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=2, d_e=136, k_m=2),
    "ub_f32_wgrad": P.small(b=8, l=77, d=136, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=4, d_e=136, k_m=2),
    "ub_f32_du": P.small(b=64, l=264, d=136, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=2, d_e=24, k_m=1),
    "ub_wgrad": P.small(b=8, l=77, d=136, n_a=2, d_h=8, m=1, c=1, k_a=1, n_m=4, d_e=136, k_m=2, dtype=BF),
    # Z and dH in one launch: large tiles with waves that straddle experts; no room for the gate's sums: two launches
    "ub_dual_large": P.small(b=44, l=150, d=40, n_a=1, d_h=8, m=1, c=1, k_a=1, n_m=3, d_e=88, k_m=3, dtype=BF),
    "ub_dual_no_room": P.small(b=128, l=1000, d=8, n_a=1, d_h=8, m=1, c=1, k_a=1, n_m=1, d_e=8, k_m=1, dtype=BF),
    # the same on the 32-grid, every tile shape, K-steps of 64 and of 32, rows and columns that end inside a tile
    "ub_dual_128x64": P.small(b=44, l=224, d=64, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=3, d_e=160, k_m=2, dtype=BF),
    "ub_dual_128x32": P.small(b=44, l=224, d=96, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=3, d_e=160, k_m=2, dtype=BF),
    "ub_dual_32": P.small(b=2, l=96, d=32, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=3, d_e=96, k_m=2, dtype=BF),
    "ub_dual_64x64": P.small(b=2, l=96, d=64, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=3, d_e=96, k_m=2, dtype=BF),
    "ub_dual_64x128": P.small(b=40, l=224, d=64, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=3, d_e=96, k_m=2, dtype=BF),
}
P.BWD_CONFIGS.update(UOME_BWD)
SMHA_BWD = {
    "sb_lp7": P.small(b=3, l=105, d=72, n_a=4, d_h=40, m=15, c=4, k_a=3, n_m=2, d_e=32, k_m=1, dtype=BF),
    "sb_dh120": P.small(b=2, l=198, d=40, n_a=3, d_h=120, m=6, c=3, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
    "sb_f32_dh128": P.small(b=1, l=200, d=64, n_a=2, d_h=128, m=4, c=3, k_a=1, n_m=2, d_e=32, k_m=1),
    "sb_f32_b130": P.small(b=130, l=8, d=16, n_a=2, d_h=8, m=4, c=2, k_a=1, n_m=2, d_e=32, k_m=1),
    # 72 rows in four waves of at most a tile each, however many blocks; longer units: two waves from 512 32-row blocks on, four below
    # (one from 1024 on: test_gpu_attention_one_tile.py)
    "sb_f32_ks1": P.small(b=128, l=72, d=16, n_a=4, d_h=16, m=2, c=2, k_a=4, n_m=2, d_e=32, k_m=1),
    "sb_f32_ks2": P.small(b=64, l=130, d=16, n_a=2, d_h=64, m=2, c=2, k_a=2, n_m=2, d_e=32, k_m=1),
    "sb_f32_ks4": P.small(b=2, l=300, d=24, n_a=3, d_h=32, m=10, c=9, k_a=2, n_m=2, d_e=32, k_m=1),
    # 128-column heads, weight gradients of 8 experts in 8 parts (bf16: 128x128 tiles)
    "sb_f32_wgrad": P.small(b=32, l=72, d=40, n_a=8, d_h=128, m=9, c=8, k_a=2, n_m=2, d_e=32, k_m=1),
    "sb_wgrad": P.small(b=32, l=72, d=40, n_a=8, d_h=120, m=9, c=8, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
    # 32-grid: dO on 128-row tiles with K-steps of 64 and of 32
    "sb_do_128x64": P.small(b=65, l=512, d=64, n_a=4, d_h=64, m=8, c=4, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
    "sb_do_128x32": P.small(b=65, l=512, d=96, n_a=4, d_h=64, m=8, c=4, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
    # one wave group per own block with two streamed tiles (2048 blocks); d_x of 32-row patches as a launch of its own
    "sb_one_group": P.small(b=128, l=128, d=32, n_a=17, d_h=32, m=4, c=4, k_a=4, n_m=2, d_e=32, k_m=1, dtype=BF),
    # one key per query: dS is exactly zero
    "sb_lp1_c1": P.small(b=2, l=6, d=8, n_a=2, d_h=8, m=6, c=1, k_a=1, n_m=2, d_e=8, k_m=1, dtype=BF),
}
P.SMHA_BWD_CONFIGS.update(SMHA_BWD)


@pytest.mark.parametrize("name", list(UOME_BWD))
@pytest.mark.parametrize("flags", [0, R | GE])
def test_uome_backward_odd_sizes(name, flags):
    P.test_uome_backward_parity(name, flags)


@pytest.mark.parametrize("name", list(SMHA_BWD))
@pytest.mark.parametrize("flags,rope_dim,pad_frac", [(0, 0, 0.0), (CA | R | GE | GP, 8, 0.2)])
def test_smha_backward_odd_sizes(name, flags, rope_dim, pad_frac):
    P.run_smha_backward(name, flags, rope_dim, pad_frac=pad_frac)


@pytest.mark.parametrize("name", [n for n in SMHA_BWD if n.startswith("sb_f32")])
def test_smha_backward_f32_logits_of_order_one(name, monkeypatch):
    order_one_logits(monkeypatch)
    P.run_smha_backward(name, R | GE | GP, 0)


# data selection on the 32-grid: every tile of dH (256, 128 and 64 rows, wave tiles of 64 and of 32 columns) and d_u and
# the weight gradients as launches of their own (64-row patches; 256-row weight-gradient tiles)
DS_BWD = {
    "dsb_256x256x64": P.small(b=64, l=192, d=768, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=4, d_e=256, k_m=4, m_m=6, c_m=5, dtype=BF),
    "dsb_128x256x32": P.small(b=48, l=192, d=96, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=4, d_e=256, k_m=4, m_m=6, c_m=5, dtype=BF),
    "dsb_128x128x64": P.small(b=20, l=192, d=64, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=5, d_e=160, k_m=4, m_m=6, c_m=5, dtype=BF),
    "dsb_128x128x32": P.small(b=20, l=192, d=96, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=5, d_e=160, k_m=4, m_m=6, c_m=5, dtype=BF),
    "dsb_64x128x64": P.small(b=10, l=192, d=64, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=5, d_e=160, k_m=4, m_m=6, c_m=5, dtype=BF),
    "dsb_own_launches": P.small(b=32, l=512, d=192, n_a=2, d_h=32, m=2, c=1, k_a=1, n_m=16, d_e=160, k_m=8, m_m=8, c_m=4, dtype=BF),
}
P.DS_BWD_CONFIGS.update(DS_BWD)


@pytest.mark.parametrize("name", list(DS_BWD))
@pytest.mark.parametrize("flags", [0, R | GE | GP])
def test_uome_data_selection_backward_tiles(name, flags):
    P.test_uome_data_selection_backward_parity(name, flags)


# --------------------------------------------------------------------------- router backward
ROUTE_BWD = {
    # one sample and 8 samples or fewer per d_x thread, columns below one 16-tile, one patch
    "rb_one": P.small(b=1, l=3, d=8, n_a=1, d_h=8, m=1, c=1, k_a=1, n_m=1, d_e=8, k_m=1),
    "rb_d24": P.small(b=5, l=130, d=24, n_a=3, d_h=8, m=10, c=2, k_a=2, n_m=2, d_e=8, k_m=1, dtype=BF),
    # samples shared by eight lanes of dW_E (b >= 8), second expert tile, two column slices, the last one short
    "rb_n17": P.small(b=9, l=65, d=264, n_a=17, d_h=8, m=65, c=2, k_a=2, n_m=2, d_e=8, k_m=1, dtype=BF),
    "rb_f32_n32": P.small(b=13, l=66, d=264, n_a=32, d_h=8, m=33, c=2, k_a=2, n_m=2, d_e=8, k_m=1),
    # four samples per d_x thread, the last group of one; chunks of more than one tile
    "rb_b9_long": P.small(b=9, l=2100, d=256, n_a=4, d_h=8, m=70, c=2, k_a=2, n_m=2, d_e=8, k_m=1, dtype=BF),
    # eight samples per d_x thread (b > 4, n <= 16, W_E of 3 * 2^23 elements and more), the last group of one or three
    "rb_b9_eight": P.small(b=9, l=2100, d=1024, n_a=12, d_h=8, m=70, c=2, k_a=2, n_m=2, d_e=8, k_m=1, dtype=BF),
    "rb_f32_eight": P.small(b=11, l=3300, d=640, n_a=12, d_h=8, m=60, c=2, k_a=2, n_m=2, d_e=8, k_m=1),
    # 2048 columns: eight slices
    "rb_d2048": P.small(b=2, l=40, d=2048, n_a=5, d_h=8, m=8, c=2, k_a=2, n_m=2, d_e=8, k_m=1, dtype=BF),
}
P.EDGE_CONFIGS.update(ROUTE_BWD)


@pytest.mark.parametrize("name", list(ROUTE_BWD))
@pytest.mark.parametrize("routers", ["both", "expert", "data"])
def test_route_backward_odd_sizes(name, routers, monkeypatch):
    """A call with one router only leaves the other one's outputs alone and adds its own part to d_x."""
    if routers == "both":
        P.test_route_backward_parity(name)
        return
    print(f"route backward {name} {routers}", flush=True)
    monkeypatch.setenv("UOE_STREAM_ONCE_MIN_BYTES", "0")  # the hinted accesses as well
    cfg = P.get_cfg(name)
    inp = synth.make_inputs(cfg, w_std=0.02)
    inp.a_w_expert = inp.a_w_expert * P.np.float32(0.25)
    e, d = (inp.a_w_expert, None) if routers == "expert" else (None, inp.a_w_b)
    wa = None if d is None else inp.a_w_a
    ref = P.oracle.route(inp.x, cfg.n_a, cfg.k_a, cfg.m, cfg.c, inp.a_w_expert, inp.a_w_b, inp.a_w_a, None, None)
    ge, gp = ref.expert_gate.astype("float32"), ref.patch_gate.astype("float32")
    d_ge, d_gp = synth.make_gate_grads(cfg, cfg.n_a, cfg.m)
    d_x0 = synth.make_upstream_grad(cfg)
    dev = P.DeviceLayer(inp, R, R)
    f32 = lambda a: P.to_device(a, synth.F32, dev.device)
    d_x = P.to_device(d_x0, cfg.dtype, dev.device)
    d_we, d_wb, d_wa = (P.torch.full_like(t, 7.0) for t in (dev.a_w_expert, dev.a_w_b, dev.a_w_a))
    ws = P.torch.empty(B.route_backward_workspace_bytes(dev.smha), dtype=P.torch.uint8, device=dev.device)
    B.route_backward(dev.smha, dev.x, None if e is None else dev.a_w_expert, None if d is None else dev.a_w_b,
                     None if d is None else dev.a_w_a, f32(ge), f32(gp), f32(d_ge), f32(d_gp), d_x, d_we, d_wb, d_wa, ws)
    P.torch.cuda.synchronize()
    want = P.oracle.route_backward(inp.x, e, d, wa, ge, gp, d_ge, d_gp)
    errs = [P.scaled_err(P.to_host(d_x), d_x0.astype("float64") + want.d_x)]
    if d is None:
        errs.append(P.grad_err(P.to_host(d_we), want.d_w_expert))
        assert bool((d_wb == 7.0).all()) and bool((d_wa == 7.0).all())
    else:
        errs += [P.grad_err(P.to_host(d_wb).T, want.d_w_b.T), P.grad_err(P.to_host(d_wa).T, want.d_w_a.T)]
        assert bool((d_we == 7.0).all())
    assert max(errs) <= P.TOL[cfg.dtype], errs
