"""Both layers of the UoME block in one launch with the expert selection in its workgroups (uoe_layer_forward) against the selection as a launch and the
block's own call: the same bits, for every number of 32-column tiles, eight and four waves, last workgroups with waves that have no token, last
stages of 32 hidden columns.  Then infinities and NaN in that launch against the two layers' own calls."""
import pytest
import torch

import test_gpu_parity as P
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth
from paper_2503_02495_amd.harness import DeviceLayer

pytestmark = pytest.mark.gpu

SMHA = dict(n_a=2, d_h=32, m=2, c=1, k_a=1, dtype=synth.BF16)
R, GE = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT
CASES = [  # b, l, d, n, k, d_e: tokens fill 0.6 of a round of 256-row workgroups (eight waves), or 0.75 of 128-row ones (four; up to 224 columns)
    (160, 250, 32, 3, 1, 32), (10, 4098, 64, 4, 3, 32), (16, 2560, 96, 5, 2, 96), (160, 256, 128, 4, 2, 64), (41, 1000, 160, 4, 3, 160),
    (10, 4098, 192, 3, 3, 32), (20, 2048, 224, 4, 1, 224), (10, 4098, 256, 9, 4, 32),
    (24, 1026, 32, 32, 4, 32), (25, 1000, 64, 4, 1, 32), (200, 128, 96, 3, 2, 96), (25, 1000, 128, 5, 2, 32), (24, 1026, 160, 4, 2, 32),
    (128, 196, 192, 6, 3, 96), (200, 128, 224, 3, 2, 96)]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_selection_in_the_launch_of_both_layers(case):
    b, l, d, n, k, d_e = case
    cfg = P.small(b=b, l=l, d=d, n_m=n, k_m=k, d_e=d_e, router_noise=True, **SMHA)
    inp = synth.make_inputs(cfg)
    one, other = (DeviceLayer(inp, P.R | P.GE | P.GP, P.R | P.GE) for _ in range(2))
    one.layer_forward()
    for run in (other.route_a, other.smha_forward, other.route_m, other.uome_forward):
        run()
    torch.cuda.synchronize()
    for key in ("m_expert_idx", "m_expert_gate", "out"):
        got, want = getattr(one, key), getattr(other, key)
        same = torch.int16 if got.element_size() == 2 else torch.int32
        assert torch.equal(got.view(same), want.view(same)), key


@pytest.mark.parametrize("case", [(160, 250, 32, 3, 1, 32), (41, 1000, 160, 4, 3, 160), (10, 4096, 256, 8, 4, 32), (24, 1024, 32, 4, 3, 32)],
                         ids=lambda c: "x".join(map(str, c)))
def test_infinities_and_nan(case):
    b, l, d, n, k, d_e = case
    gen = torch.Generator(device="cuda").manual_seed(d)
    draw = lambda *s, std: (torch.randn(s, generator=gen, device="cuda") * std).to(torch.bfloat16)
    u, a_in, a_out = draw(b, l, d, std=1.0), draw(n, d, d_e, std=0.1), draw(n, d_e, d, std=0.1)
    idx = torch.arange(1, k + 1, device="cuda", dtype=torch.int32).clamp(max=n - 1).repeat(b, 1).contiguous()   # expert 0 is not selected
    gate = torch.rand(b, n, generator=gen, device="cuda")
    inf, nan = float("inf"), float("nan")
    u[0, 3, 5], u[1, 7, 2], u[1, 40, 0], u[2, l - 1, d - 1], u[3, 100, 1] = nan, inf, -inf, inf, 3e38
    a_in[0], a_out[0, 1] = nan, inf
    a_out[1, d_e - 1, 3] = inf
    a_in[1, 2, 0] = 60.0
    desc = B.block_desc(b, l, d, n, k, 1, 1, d_e, B.BF16, R | GE)
    ws = torch.empty(B.workspace_bytes(None, desc), dtype=torch.uint8, device="cuda")
    out, want = (torch.zeros(b, l, d, device="cuda", dtype=torch.bfloat16) for _ in range(2))
    hidden = torch.empty(b, l, k * d_e, device="cuda", dtype=torch.bfloat16)
    B.uome_forward(desc, u, a_in, a_out, idx, gate, None, None, out, ws)
    B.uome_up(desc, u, a_in, idx, gate, hidden)
    B.uome_down(desc, hidden, a_out, u, idx, want)
    torch.cuda.synchronize()
    got, ref = out.float(), want.float()
    assert not torch.isfinite(ref).all() and torch.isfinite(ref[4:, :, 4:]).any()
    assert torch.equal(got.isnan(), ref.isnan())
    assert torch.equal(torch.where(got.isinf(), got, torch.zeros_like(got)), torch.where(ref.isinf(), ref, torch.zeros_like(ref)))
    # one bf16 step of the product and one of the result (the layers' own calls: another order of fp32 sums), and that order's error beside cancelling terms
    ok = torch.isfinite(ref) & torch.isfinite(u.float()).all(-1, keepdim=True) & (u.float().abs().amax(-1, keepdim=True) < 100)
    g, r, x = got[ok], ref[ok], u.float()[ok]
    assert ok.any() and ((g - r).abs() <= (2.0 ** -7) * ((r - x).abs() + r.abs()) + 1e-3 * r.abs().max()).all()
