"""The layer's backward pass, where a block's last launches share the routers' (the reduction of the weight gradients, the gate gradients,
the data router's first step), against the blocks' and routers' calls one by one: the same bits, with and without the paired
contractions, in both storage types, on and off the 32-grid, with data selection, and with reductions of ragged tiles."""
import pytest
import torch

import test_gpu_parity as P
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth
from paper_2503_02495_amd.harness import DeviceLayer, to_device

pytestmark = pytest.mark.gpu

BF = dict(dtype=synth.BF16)
CONFIGS = {
    # both blocks' contractions paired; 96-wide widths: ragged 64 x 64 tiles of the reduction
    "paired": P.small(b=3, l=128, d=96, n_a=4, d_h=64, m=4, c=2, k_a=2, n_m=4, d_e=192, k_m=2, **BF),
    "paired_data_selection": P.small(b=2, l=128, d=96, n_a=4, d_h=32, m=4, c=2, k_a=2, n_m=4, d_e=96, k_m=2, m_m=4, c_m=2, **BF),
    "neither_paired": P.small(b=2, l=64, d=640, n_a=32, d_h=32, m=2, c=1, k_a=2, n_m=4, d_e=64, k_m=2, **BF),
    "one_of_each": P.small(b=1, l=32, d=32, n_a=1, d_h=32, m=1, c=1, k_a=1, n_m=1, d_e=32, k_m=1, **BF),
    "off_grid": P.small(b=5, l=70, d=72, n_a=3, d_h=40, m=5, c=2, k_a=2, n_m=3, d_e=40, k_m=2, **BF),
    "off_grid_f32": P.small(b=128, l=14, d=40, n_a=3, d_h=8, m=2, c=1, k_a=1, n_m=3, d_e=72, k_m=3),
    "f32_long_units": P.small(b=2, l=512, d=64, n_a=2, d_h=64, m=2, c=2, k_a=2, n_m=2, d_e=64, k_m=1),
}


@pytest.mark.parametrize("name", list(CONFIGS))
def test_layer_backward_against_its_calls(name):
    cfg = CONFIGS[name]
    inp = synth.make_inputs(cfg)
    dev = DeviceLayer(inp, P.R | P.GE | P.GP, P.R | P.GE | (P.GP if cfg.m_m > 1 else 0))
    for run in (dev.route_a, dev.smha_forward, dev.route_m, dev.uome_forward):
        run()
    d_out = to_device(synth.make_upstream_grad(cfg), cfg.dtype, dev.device)
    got = {k: v.clone() for k, v in dev.layer_backward(d_out, u=dev.u).items() if v is not None}

    want = {k: torch.full_like(v, float("nan")) for k, v in got.items()}
    um = B.block_desc(cfg.b, cfg.l, cfg.d, cfg.n_m, cfg.k_m, cfg.m_m, cfg.c_m, cfg.d_e, dev.uome.dtype, dev.uome.flags)
    ws = torch.empty(max(B.route_backward_workspace_bytes(um), B.route_backward_workspace_bytes(dev.smha)), dtype=torch.uint8, device=dev.device)
    d_u, d_a_in, d_a_out, d_gate, *d_pgate = dev.uome_backward(d_out)
    want["d_a_in"], want["d_a_out"] = d_a_in, d_a_out
    B.route_backward(um, dev.u, dev.m_w_expert, dev.m_w_b, dev.m_w_a, dev.m_expert_gate, dev.m_patch_gate, d_gate, d_pgate[0] if d_pgate else None,
                     d_u, want["d_m_w_expert"], want.get("d_m_w_b"), want.get("d_m_w_a"), ws)
    d_x, want["d_wq"], want["d_wk"], want["d_wv"], want["d_wo"], d_ge, d_gp = dev.smha_backward(d_u)
    B.route_backward(dev.smha, dev.x, dev.a_w_expert, dev.a_w_b, dev.a_w_a, dev.a_expert_gate, dev.a_patch_gate, d_ge, d_gp, d_x, want["d_a_w_expert"],
                     want["d_a_w_b"], want["d_a_w_a"], ws)
    want["d_x"] = d_x
    torch.cuda.synchronize()
    for k, v in got.items():
        same = torch.int16 if v.element_size() == 2 else torch.int32
        assert torch.isfinite(v.float()).all(), k
        assert torch.equal(v.view(same), want[k].view(same)), k
