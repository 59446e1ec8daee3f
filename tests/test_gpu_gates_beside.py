"""The gate gradient of the expert-selection MLP block off the 32-grid and in fp32, which runs in workgroups behind d_u's tiles: one
shape per tile of that contraction (128, 256 or 512 threads), against fp64."""
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu

N, K, D_E = 3, 2, 40
SHAPES = {  # b, l, d, type; the tile of d_u
    "bf16_32x128": (3, 20, 72, torch.bfloat16),
    "bf16_64x128": (3, 70, 72, torch.bfloat16),
    "bf16_128x128": (64, 250, 264, torch.bfloat16),
    "f32_32x64": (3, 70, 72, torch.float32),
    "f32_64x64_exact": (40, 100, 72, torch.float32),
    "f32_64x64": (70, 100, 72, torch.float32),
    "f32_64x128": (128, 256, 128, torch.float32),
    "f32_128x128": (256, 256, 128, torch.float32),
}


@pytest.mark.parametrize("name", list(SHAPES))
def test_gate_gradient(name):
    b, l, d, dtype = SHAPES[name]
    gen = torch.Generator().manual_seed(7)

    def rand(*shape, scale=1.0):
        return (torch.randn(*shape, generator=gen) * scale).to(dtype).cuda()

    u, d_out = rand(b, l, d), rand(b, l, d)
    a_in, a_out = rand(N, d, D_E, scale=d ** -0.5), rand(N, D_E, d, scale=d ** -0.5)
    idx = torch.stack([torch.randperm(N, generator=gen)[:K].sort().values for _ in range(b)]).to(torch.int32).cuda()
    gate = torch.rand(b, N, generator=gen).cuda()
    desc = B.block_desc(b, l, d, N, K, 1, 1, D_E, B.BF16 if dtype == torch.bfloat16 else B.F32, B.FLAG_RESIDUAL | B.FLAG_GATE_EXPERT)
    d_gate = torch.full_like(gate, float("nan"))
    ws = torch.empty(B.uome_backward_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    B.uome_backward(desc, u, a_in, a_out, idx, gate, None, None, d_out, torch.empty_like(u), torch.empty_like(a_in), torch.empty_like(a_out), d_gate, None, ws)
    torch.cuda.synchronize()
    for s in range(b):
        chosen = idx[s].tolist()
        for i in range(N):
            if i not in chosen:
                assert d_gate[s, i] == 0
                continue
            z = u[s].cpu().double() @ a_in[i].cpu().double()
            terms = d_out[s].cpu().double() @ a_out[i].cpu().double().T * z * torch.sigmoid(z)
            # a term's two sums of d products are off by about sqrt(d) fp32 roundings of 2^-24, 2^-20 for d = 264; four times that for both, the
            # sigmoid and the sums of terms
            assert abs(d_gate[s, i].cpu().double() - terms.sum()) <= 2.0 ** -18 * terms.abs().sum(), (s, i)
