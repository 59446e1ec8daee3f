"""The gate gradient of the expert-selection MLP block off the 32-grid and in fp32, which runs in workgroups behind d_u's tiles: one
shape per tile of that contraction (128, 256 or 512 threads), against fp64, and the order of its sums."""
import numpy as np
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


# b, l, d, d_e, type, rows a partial sum is of; d_u's tiles have 128, 512 and 256 threads
ORDERED = [(1, 190, 72, 1040, torch.float32, 32), (64, 500, 64, 1032, torch.bfloat16, 64), (1, 190, 72, 1032, torch.bfloat16, 32)]


@pytest.mark.parametrize("b,l,d,d_e,dtype,rows", ORDERED)
def test_order_of_the_sums(b, l, d, d_e, dtype, rows):
    """256 strided subsets, then halves, whatever the number of threads.  Z is 128 (its SiLU too), and of the rows and columns of a partial sum one
    each is not zero: the sums' terms are exact, and pairs of 2^20 that cancel in part of the orders only show any other."""
    rng = np.random.default_rng(l + 1)
    blocks, groups = -(-l // rows), d_e // 8
    alpha = np.array([1.0, -0.5, 2.0, -1.0, 0.25, -2.0, 0.5, -0.25][:blocks], np.float32)
    beta = rng.integers(-16, 17, groups).astype(np.float32) / 16
    at = rng.permutation(groups)[:groups // 4 * 2]
    beta[at[0::2]], beta[at[1::2]] = 2.0 ** 20, -2.0 ** 20
    terms = (alpha[:, None] * beta * 128).reshape(-1).astype(np.float32)

    def by(subsets):
        red = np.zeros(subsets, np.float32)
        for i, t in enumerate(terms):
            red[i % subsets] += t
        while len(red) > 1:
            red = red[:len(red) // 2] + red[len(red) // 2:]
        return red[0]

    want = by(256)
    assert want != by(128 if dtype == torch.float32 else 512)
    u, d_out = torch.zeros(b, l, d), torch.zeros(b, l, d)
    a_in, a_out = torch.zeros(2, d, d_e), torch.zeros(2, d_e, d)
    u[:, :, 0] = 1
    a_in[:, 0] = 128
    d_out[:, ::rows, 0] = torch.from_numpy(alpha)
    a_out[:, ::8, 0] = torch.from_numpy(beta)
    u, d_out, a_in, a_out = (t.to(dtype).cuda() for t in (u, d_out, a_in, a_out))
    idx = torch.zeros(b, 1, dtype=torch.int32, device="cuda")
    gate = torch.ones(b, 2, device="cuda")
    desc = B.block_desc(b, l, d, 2, 1, 1, 1, d_e, B.BF16 if dtype == torch.bfloat16 else B.F32, B.FLAG_GATE_EXPERT)
    d_gate = torch.full_like(gate, float("nan"))
    ws = torch.empty(B.uome_backward_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    B.uome_backward(desc, u, a_in, a_out, idx, gate, None, None, d_out, torch.empty_like(u), torch.empty_like(a_in), torch.empty_like(a_out), d_gate, None, ws)
    torch.cuda.synchronize()
    assert (d_gate[:, 0].cpu().numpy() == want).all(), (d_gate[0, 0].item(), want)
    assert (d_gate[:, 1] == 0).all()
