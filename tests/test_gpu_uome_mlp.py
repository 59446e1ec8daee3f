"""Both layers of the expert-selection UoME block in one launch (bf16, d <= 256) against its two layers' own calls: every number of 32-column
tiles, last stages of 32 hidden columns, stages of two experts, ragged last workgroups, four and eight waves, without residual or gate.

Both round h and the product to bf16 and add the residual in fp32; they differ in the order of fp32 sums, so an element is the same or, where a
sum crosses a rounding boundary, one bf16 step of the product (2^-8 of it) and one of the result apart."""
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu

R, GE = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT
CASES = [  # b, l, d, n, k, d_e, flags; tokens fill 0.6 of a round of 256-row workgroups (eight waves), or 0.75 of 128-row ones (four)
    (160, 250, 32, 3, 1, 32, R | GE),
    (10, 4096, 64, 4, 3, 32, R | GE),
    (16, 2560, 96, 5, 2, 96, R | GE),
    (160, 256, 128, 4, 2, 64, GE),
    (41, 1000, 160, 4, 3, 160, R),
    (10, 4097, 192, 3, 3, 32, R | GE),
    (20, 2048, 224, 4, 1, 224, R | GE),
    (10, 4096, 256, 8, 4, 32, R | GE),
    (64, 641, 256, 2, 1, 416, 0),
    (128, 196, 192, 6, 3, 96, R | GE),
    (24, 1024, 32, 4, 4, 64, R | GE),
    (25, 1000, 160, 4, 2, 32, R | GE),
    (200, 128, 224, 3, 2, 96, GE),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(map(str, c)))
def test_both_layers_in_one_launch(case):
    b, l, d, n, k, d_e, flags = case
    gen = torch.Generator(device="cuda").manual_seed(l + d)
    draw = lambda *s, std: (torch.randn(s, generator=gen, device="cuda") * std).to(torch.bfloat16)
    u, a_in, a_out = draw(b, l, d, std=1.0), draw(n, d, d_e, std=0.1), draw(n, d_e, d, std=0.1)
    idx = torch.argsort(torch.rand(b, n, generator=gen, device="cuda"), 1)[:, :k].sort(1)[0].to(torch.int32).contiguous()
    gate = torch.rand(b, n, generator=gen, device="cuda")
    desc = B.block_desc(b, l, d, n, k, 1, 1, d_e, B.BF16, flags)
    ws = torch.empty(B.workspace_bytes(None, desc), dtype=torch.uint8, device="cuda")
    out, want = (torch.full((b, l, d), float("nan"), device="cuda", dtype=torch.bfloat16) for _ in range(2))
    hidden = torch.empty(b, l, k * d_e, device="cuda", dtype=torch.bfloat16)
    B.uome_forward(desc, u, a_in, a_out, idx, gate, None, None, out, ws)
    B.uome_up(desc, u, a_in, idx, gate, hidden)
    B.uome_down(desc, hidden, a_out, u, idx, want)
    torch.cuda.synchronize()
    got, ref = out.float(), want.float()
    product = (ref - u.float()).abs() if flags & R else ref.abs()
    step = (2.0 ** -7) * (product + ref.abs()) + 1e-3 * ref.abs().max()
    assert torch.isfinite(got).all()
    assert ((got - ref).abs() <= step).all()
    assert (got != ref).float().mean() < 0.02
