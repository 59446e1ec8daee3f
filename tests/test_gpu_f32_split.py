"""The fp32 contractions on split bf16 products: K one step past the fp32 instruction's range and inside a step, segments of a
K-step and less, values at the ends of the range, every tile and operand layout, and operands that are not finite (or overflow in the
split: every tile's second contraction).  The fp32 attention, and what the bf16 one off the 32-grid does with such values."""
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu


def make(b, l, d, n, k, d_e, seed=5):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    idx = torch.stack([torch.randperm(n, generator=g, device="cuda")[:k].sort().values for _ in range(b)]).int().contiguous()
    return rnd(b, l, d), 0.1 * rnd(n, d, d_e), 0.1 * rnd(n, d_e, d), idx


def down(x, w_out, idx, u):
    b, l, d = u.shape
    n, d_e, _ = w_out.shape
    out = torch.empty_like(u)
    B.uome_down(B.block_desc(b, l, d, n, idx.shape[1], 1, 1, d_e, B.F32, 0), x, w_out, u, idx, out)
    return out


def down64(x, w_out, idx):
    w = torch.cat([w_out.double()[idx[:, s].long()] for s in range(idx.shape[1])], 1)
    return torch.bmm(x.double(), w.contiguous())


@pytest.mark.parametrize("b,l,d,k,d_e", [(2, 40, 72, 2, 64), (2, 40, 72, 1, 136), (3, 33, 40, 3, 56), (2, 129, 200, 2, 232),
                                         (16, 200, 264, 2, 96), (9, 700, 520, 1, 264), (1, 65, 1032, 4, 1000)])
def test_contraction_against_fp64(b, l, d, k, d_e):
    """Relative error of a K-term fp32 sum: sqrt(K) roundings of 2^-25 of the sum at random, K <= 4000: 2e-6; a part of an
    operand lost (2^-16) or a product of parts left out (2^-17) would show."""
    print(f"fp32 contraction b={b} l={l} d={d} k={k} d_e={d_e}", flush=True)
    u, _, w_out, idx = make(b, l, d, 4, k, d_e)
    x = torch.randn((b, l, k * d_e), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda")
    got, want = down(x, w_out, idx, u).double(), down64(x, w_out, idx)
    assert (got - want).norm() <= 2e-6 * want.norm()
    # the mean over many outputs: a one-sided rounding of 2^-25 of every output's magnitude would be sqrt(outputs) times it
    bias = (got - want).mean().abs() / want.pow(2).mean().sqrt()
    assert bias <= 2e-8 + 4e-7 / want.numel() ** 0.5, bias


def test_operands_that_are_not_finite():
    """A row with one infinity gives the infinities of the fp32 product (no NaN where the other factor is finite), a NaN its
    row, a value past bf16's largest a finite row, and the other rows of the same tiles do not notice."""
    b, l, d, k, d_e = 1, 70, 96, 2, 128
    u, _, w_out, idx = make(b, l, d, 4, k, d_e)
    x = torch.randn((b, l, k * d_e), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda")
    clean = down(x, w_out, idx, u)
    x[0, 3, 17], x[0, 40, 5], x[0, 66, 200] = float("inf"), float("nan"), 3.4e38
    w_out[w_out.abs() < 1e-3] = 1e-3
    got, want = down(x, w_out, idx, u), down64(x, w_out, idx)
    col = torch.cat([w_out[idx[0, s].long()] for s in range(k)], 0)[17]
    assert torch.equal(got[0, 3], torch.where(col > 0, float("inf"), -float("inf")))
    assert got[0, 40].isnan().all()
    assert ((got[0, 66].double() - want[0, 66]).norm() <= 2e-6 * want[0, 66].norm())
    rest = [r for r in range(l) if r not in (3, 40, 66)]
    assert (got[0, rest].double() - want[0, rest]).norm() <= 2e-6 * want[0, rest].norm() and clean.isfinite().all()


def test_attention_values_that_are_not_finite():
    """One token's v overflows to infinity in one column (probabilities of 1 are one part and two zeros): the block's output
    is the infinity that W^o carries on, as with fp32 products."""
    l, d, d_h = 48, 168, 40
    g = torch.Generator(device="cuda").manual_seed(9)
    x = torch.randn((1, l, d), generator=g, device="cuda")
    x[0, :, 0] = 0.0
    x[0, 7, 0] = 1e30
    wq, wk, wv = (torch.zeros((1, d, d_h), device="cuda") for _ in range(3))
    wv[0, 1:] = 0.1 * torch.randn((d - 1, d_h), generator=g, device="cuda")
    wv[0, 0, 3] = 1e10
    wo = torch.where(torch.rand((1, d_h, d), generator=g, device="cuda") < 0.5, -0.5, 0.5)
    blk = B.block_desc(1, l, d, 1, 1, 1, 1, d_h, B.F32, 0)
    zero, one = torch.zeros((1, 1), dtype=torch.int32, device="cuda"), torch.ones((1, 1), device="cuda")
    out = torch.empty_like(x)
    ws = torch.empty(B.workspace_bytes(blk, None), dtype=torch.uint8, device="cuda")
    B.smha_forward(blk, x, wq, wk, wv, wo, zero, one, zero.reshape(1, 1, 1), one.reshape(1, 1, 1), out, ws)
    want = torch.where(wo[0, 3] > 0, float("inf"), -float("inf")).expand(l, d)
    assert torch.equal(out[0], want)


def one_unit(x, wq, wk, wv, wo):
    """The SMHA block without residual and gates where one expert takes the whole sample."""
    b, l, d = x.shape
    d_h = wq.shape[2]
    blk = B.block_desc(b, l, d, 1, 1, 1, 1, d_h, B.F32 if x.dtype == torch.float32 else B.BF16, 0)
    zero, one = torch.zeros((b, 1), dtype=torch.int32, device="cuda"), torch.ones((b, 1), device="cuda")
    out = torch.empty_like(x)
    ws = torch.empty(B.workspace_bytes(blk, None), dtype=torch.uint8, device="cuda")
    B.smha_forward(blk, x, wq, wk, wv, wo, zero, one, zero.reshape(b, 1, 1), one.reshape(b, 1, 1), out, ws)
    return out


@pytest.mark.parametrize("l", [20, 64, 100, 300])
@pytest.mark.parametrize("v_size", [1.0, 1e-36])
def test_fp32_attention_keeps_the_bits_of_small_values(l, v_size):
    """fp32 heads whose v are near the bottom of the range: the bits of a sum of l terms, as for v of order one (2^-25 of the
    sum per rounding, some l of them at random, three products in a row: 2e-6)."""
    d, d_h = 96, 40
    g = torch.Generator(device="cuda").manual_seed(11)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, wq, wk, wv, wo = rnd(2, l, d), 0.1 * rnd(1, d, d_h), 0.1 * rnd(1, d, d_h), 0.1 * rnd(1, d, d_h), rnd(1, d_h, d)
    got = one_unit(x, wq, wk, (v_size * wv).contiguous(), wo).double()
    q, k, v = (x.double() @ w[0].double() for w in (wq, wk, v_size * wv))
    p = torch.softmax(torch.bmm(q, k.transpose(1, 2).contiguous()) / d_h ** 0.5, -1)
    want = torch.bmm(p, v) @ wo[0].double()
    assert (got - want).norm() <= 2e-6 * want.norm()


@pytest.mark.parametrize("rows", [30, 128, 200])
def test_bf16_attention_off_the_grid_with_small_values(rows):
    """v of 1e-36 in bf16 heads of 40: the probabilities' lowest parts times v are below the normal numbers, o is not (v, o and the
    output are rounded to bf16 once each: 1e-2)."""
    d, d_h = 96, 40
    g = torch.Generator(device="cuda").manual_seed(13)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, wq, wk, wv, wo = (t.bfloat16() for t in (rnd(1, rows, d), 0.1 * rnd(1, d, d_h), 0.1 * rnd(1, d, d_h), 1e-37 * rnd(1, d, d_h), rnd(1, d_h, d)))
    got = one_unit(x, wq, wk, wv, wo).double()
    q, k, v = (x[0].double() @ w[0].double() for w in (wq, wk, wv))
    want = torch.softmax(q.bfloat16().double() @ k.bfloat16().double().T / d_h ** 0.5, -1) @ v @ wo[0].double()
    assert (got[0] - want).norm() <= 1e-2 * want.norm()


@pytest.mark.parametrize("sign,first", [(1.0, False), (-1.0, True)])
def test_bf16_scores_that_overflow_before_they_are_scaled(sign, first):
    """q k of 2^128 and more times log2(e) / sqrt(d_h) is a finite fp32 number: every query takes the key with the largest score."""
    l, d, d_h = 40, 72, 40
    g = torch.Generator(device="cuda").manual_seed(12)
    x = torch.randn((1, l, d), generator=g, device="cuda")
    x[0, :, 0], x[0, :, 1] = 1.0, 1.0 + torch.arange(l, device="cuda") / 64.0
    wq, wk, wv = (torch.zeros((1, d, d_h), device="cuda") for _ in range(3))
    wq[0, 0, 0], wk[0, 1, 0] = 2.0 ** 64, sign * 2.0 ** 64
    wv[0, 2:] = 0.1 * torch.randn((d - 2, d_h), generator=g, device="cuda")
    wo = torch.randn((1, d_h, d), generator=g, device="cuda")
    x, wq, wk, wv, wo = (t.bfloat16().contiguous() for t in (x, wq, wk, wv, wo))
    got = one_unit(x, wq, wk, wv, wo).double()
    want = (x[0, 0 if first else l - 1].double() @ wv[0].double()) @ wo[0].double()
    # bf16: v and the output are rounded once each
    assert (got - want).norm() <= 1e-2 * (want.norm() * l ** 0.5)


def one_expert_grads(x, d_out, wq, wk, wv, wo, l_p, c):
    """Weight gradients of the SMHA block (expert 0 of one, the first c patches of every sample) and the same in fp64."""
    b, l, d = x.shape
    d_h, m = wq.shape[2], l // l_p
    blk = B.block_desc(b, l, d, 1, 1, m, c, d_h, B.F32, 0)
    zero, one = torch.zeros((b, 1), dtype=torch.int32, device="cuda"), torch.ones((b, 1), device="cuda")
    pidx = torch.arange(c, dtype=torch.int32, device="cuda").expand(b, 1, c).contiguous()
    got = [torch.empty_like(t) for t in (wq, wk, wv, wo)]
    ws = torch.empty(B.smha_backward_workspace_bytes(blk), dtype=torch.uint8, device="cuda")
    B.smha_backward(blk, x, B.smha_weights(None, None, None, wq, wk, wv, wo), zero, one, pidx, torch.ones((b, 1, m), device="cuda"), None, d_out,
                    torch.empty_like(x), B.smha_weight_grads(*got), torch.empty((b, 1), device="cuda"), torch.empty((b, 1, m), device="cuda"), ws)
    leaves = [w[0].double().requires_grad_(True) for w in (wq, wk, wv, wo)]
    h = x[:, :c * l_p].double()
    q, k, v = (h @ w for w in leaves[:3])
    out = torch.softmax(q @ k.transpose(1, 2) / d_h ** 0.5, -1) @ v @ leaves[3]
    return [g[0].double() for g in got], torch.autograd.grad((out * d_out[:, :c * l_p].double()).sum(), leaves)


@pytest.mark.parametrize("l_p", [1, 7, 8, 9, 14, 16, 17, 24, 32, 40])
def test_weight_gradients_of_short_patches(l_p):
    """K segments of one K-step and less, some hundred of them: every part of an expert's sum rounds some 100 times in both directions
    (3e-8 of the sum each: 1e-6 at random), and the mean over the outputs of a one-sided rounding would be that of each output."""
    b, c, d, d_h = 24, 8, 96, 64
    g = torch.Generator(device="cuda").manual_seed(21)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, d_out = rnd(b, c * l_p, d), rnd(b, c * l_p, d)
    ws = [0.1 * rnd(1, d, d_h) for _ in range(3)] + [0.1 * rnd(1, d_h, d)]
    got, want = one_expert_grads(x, d_out, *ws, l_p, c)
    for name, y, r in zip(("wq", "wk", "wv", "wo"), got, want):
        rms = r.pow(2).mean().sqrt()
        err, bias = (y - r).norm() / r.norm(), (y - r).mean().abs() / rms
        print(f"l_p={l_p} d_{name} error {err:.2e} mean {bias:.2e}", flush=True)
        assert err <= 1e-6
        # the mean of 6144 errors of 6e-7 at random: 1e-8 (one-sided: 6e-8 and more)
        assert bias <= 3e-8


@pytest.mark.parametrize("d_e,k", [(8, 16), (16, 16), (24, 12), (40, 8)])
def test_contractions_over_short_segments(d_e, k):
    """The experts' slices of K one K-step long or less."""
    u, _, w_out, idx = make(8, 130, 264, 16, k, d_e)
    x = torch.randn((8, 130, k * d_e), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda")
    got, want = down(x, w_out, idx, u).double(), down64(x, w_out, idx)
    assert (got - want).norm() <= 1e-6 * want.norm()
    assert (got - want).mean().abs() <= 5e-9 * want.pow(2).mean().sqrt()   # 274560 errors of 3e-7: 6e-10; one-sided: 1.5e-8


@pytest.mark.parametrize("x_size,w_size", [(1e-36, 1.0), (1.0, 1e-36), (1e-19, 1e-18), (1e30, 1.0), (1e19, 1e15), (1e-36, 1e36)])
def test_contractions_at_the_ends_of_the_range(x_size, w_size):
    """Operands of which the lowest parts are below the smallest normal bf16 number or the largest past the split's scale: the bits of
    operands of order one (a sum below 1e-35 is held to 2^-149 absolutely)."""
    u, _, w_out, idx = make(2, 130, 264, 4, 2, 136)
    x = torch.randn((2, 130, 272), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda") * x_size
    w_out = (w_out * w_size).contiguous()
    got, want = down(x, w_out, idx, u).double(), down64(x, w_out, idx)
    assert (got - want).norm() <= 2e-6 * want.norm() + 1e-44 * want.numel() ** 0.5


def test_experts_of_small_gates_keep_their_gradients():
    """Saturated routers give selected experts gates of 1e-38: their part of d_u is a contraction of numbers of that size."""
    u, w_in, w_out, idx = make(4, 100, 264, 4, 2, 136)
    g = torch.Generator(device="cuda").manual_seed(8)
    d_out, gate = torch.randn(u.shape, generator=g, device="cuda"), 1e-37 * (0.5 + torch.rand((4, 4), generator=g, device="cuda"))
    blk = B.block_desc(4, 100, 264, 4, 2, 1, 1, 136, B.F32, B.FLAG_GATE_EXPERT)
    d_u = torch.empty_like(u)
    ws = torch.empty(B.uome_backward_workspace_bytes(blk), dtype=torch.uint8, device="cuda")
    B.uome_backward(blk, u, w_in, w_out, idx, gate, None, None, d_out, d_u, torch.empty_like(w_in), torch.empty_like(w_out), torch.empty_like(gate),
                    None, ws)
    leaf = u.double().requires_grad_(True)
    out = 0
    for s in range(2):
        e = idx[:, s].long()
        z = torch.bmm(leaf, w_in.double()[e].contiguous())
        out = out + torch.bmm(z * torch.sigmoid(z) * gate.double().gather(1, e[:, None])[:, :, None], w_out.double()[e].contiguous())
    want, = torch.autograd.grad((out * d_out.double()).sum(), leaf)
    # factors of 1e-38 in the epilogue are subnormal in part: 2^-149 of 1e-38 each
    assert (d_u.double() - want).norm() <= 1e-5 * want.norm()


# --------------------------------------------------------------------------- tiles and layouts
def tile(km, gaps_nk, groups, rows, cols):
    """The fp32 half of tail_tile (common.h): rows and columns of the tile, and whether it is on the fp32 instruction."""
    up = lambda v, to: -(-v // to)
    n = lambda bm, bn: groups * up(rows, bm) * up(cols, bn)
    padded = lambda bm, bn: n(bm, bn) * bm * bn / (n(64, 64) * 4096)
    if km:
        if rows > 64 and n(128, 128) >= 512 and padded(128, 128) <= 1.1:
            return 128, 128, False
        return (64, 128, False) if n(64, 128) > 384 and padded(64, 128) <= 1.25 else (64, 64, False)
    if rows <= 32 or n(64, 64) <= 128:
        return 32, 64, True
    if n(64, 64) <= 256:
        return 64, 64, True
    if rows > 64 and n(128, 128) >= 512 and padded(128, 128) <= 1.1 and not gaps_nk:
        return 128, 128, False
    return (64, 128, False) if rows > 64 and n(64, 128) >= 512 and padded(64, 128) <= 1.1 else (64, 64, False)


FORWARD_TILES = [((2, 40, 72, 2, 136), (32, 64, True)), ((8, 300, 264, 1, 264), (64, 64, True)), ((12, 300, 264, 1, 264), (64, 64, False)),
                 ((9, 700, 520, 1, 264), (64, 64, False)), ((16, 500, 504, 1, 264), (64, 128, False)), ((32, 500, 504, 1, 264), (128, 128, False))]


@pytest.mark.parametrize("x_size", [1.0, 1e33])
@pytest.mark.parametrize("shape,want_tile", FORWARD_TILES)
def test_every_forward_tile(shape, want_tile, x_size):
    """x of 1e33 overflows in the split: every tile is contracted twice."""
    b, l, d, k, d_e = shape
    assert tile(False, False, b, l, d) == want_tile
    print(f"fp32 down {shape} tile {want_tile} x {x_size}", flush=True)
    u, _, w_out, idx = make(b, l, d, 4, k, d_e)
    x = torch.randn((b, l, k * d_e), generator=torch.Generator(device="cuda").manual_seed(6), device="cuda") * x_size
    got, want = down(x, w_out, idx, u).double(), down64(x, w_out, idx)
    assert (got - want).norm() <= 2e-6 * want.norm()


# b, l, d, n, k, d_e; tiles of Z / dH, of d_u, of the weight gradients
UOME_BACKWARD_TILES = [((8, 77, 200, 4, 2, 136), (64, 64, True), (32, 64, True), (64, 64, False)),
                       ((8, 200, 504, 8, 2, 248), (64, 64, True), (64, 64, True), (128, 128, False)),
                       ((32, 250, 504, 4, 2, 136), (64, 64, False), (64, 128, False), (64, 128, False)),
                       ((64, 250, 504, 2, 2, 264), (128, 128, False), (128, 128, False), (64, 128, False)),
                       ((40, 140, 136, 2, 1, 72), (64, 64, True), (64, 64, False), (64, 64, False))]


@pytest.mark.parametrize("g_size", [1.0, 1e32])
@pytest.mark.parametrize("shape,dual,du,wgrad", UOME_BACKWARD_TILES)
def test_every_uome_backward_tile(shape, dual, du, wgrad, g_size):
    """The dual launch, [n][k] right operands and weight gradients; an upstream gradient of 1e32 takes each of them through the second
    contraction (it overflows in the split)."""
    b, l, d, n, k, d_e = shape
    print(f"fp32 uome backward {shape} gradient {g_size}", flush=True)
    large, few = l > 64 and b * -(-l // 128) * -(-k * d_e // 128) >= 256, b * -(-l // 64) * -(-k * d_e // 64) <= 256
    assert dual == ((128, 128, False) if large else (64, 64, few)) and du == tile(False, False, b, l, d)
    u, w_in, w_out, idx = make(b, l, d, n, k, d_e)
    blk = B.block_desc(b, l, d, n, k, 1, 1, d_e, B.F32, 0)
    nbytes = B.uome_backward_workspace_bytes(blk)
    parts = (nbytes - 2 * b * l * k * d_e * 4) // (2 * n * d * d_e * 4)   # one chunk of samples
    assert wgrad == tile(True, False, 2 * n * parts, d_e, d)
    d_out = g_size * torch.randn(u.shape, generator=torch.Generator(device="cuda").manual_seed(8), device="cuda")
    got, gate = [torch.empty_like(t) for t in (u, w_in, w_out)], torch.ones((b, n), device="cuda")
    B.uome_backward(blk, u, w_in, w_out, idx, gate, None, None, d_out, *got, torch.empty_like(gate), None,
                    torch.empty(nbytes, dtype=torch.uint8, device="cuda"))
    leaves = [t.double().requires_grad_(True) for t in (u, w_in, w_out)]
    out = 0
    for s in range(k):
        e = idx[:, s].long()
        z = torch.bmm(leaves[0], leaves[1][e].contiguous())
        out = out + torch.bmm(z * torch.sigmoid(z), leaves[2][e].contiguous())
    for name, y, r in zip(("u", "in", "out"), got, torch.autograd.grad((out * d_out.double()).sum(), leaves)):
        err = ((y.double() - r).norm() / r.norm()).item()
        print(f"  d_{name} {err:.2e}", flush=True)
        assert err <= 2e-6


# b, patches, tokens of one, d, n, k, c, d_h; tiles of q, k, v, of the out-projection and of d_x
SMHA_TILES = [((4, 6, 9, 136, 4, 2, 3, 40), (32, 64, True), (32, 64, True), (32, 64, True)),
              ((16, 10, 20, 200, 4, 3, 6, 128), (64, 64, False), (32, 64, True), (32, 64, True)),
              ((96, 14, 14, 384, 6, 3, 4, 64), (64, 64, False), (128, 128, False), (64, 128, False)),
              ((40, 4, 120, 264, 4, 3, 3, 72), (128, 128, False), (64, 64, False), (64, 64, False)),
              ((48, 5, 110, 384, 4, 2, 4, 120), (64, 128, False), (128, 128, False), (64, 128, False))]


def patch_groups(b, l_p, m, c, d):
    """set_patch_groups (problems.h): patches in a group."""
    fit = lambda t: min(t // l_p if 2 * l_p <= t else 1, m)
    none = lambda g: (1 - c / m) ** g
    products = lambda g, t: -(-g * l_p // t) * t / g * (1 - none(g))
    g32, g128 = fit(32), min(fit(128), 32)
    many = b * -(-m // g128) * -(-d // 128) >= 512
    return g128 if l_p <= 32 and g128 > g32 and g128 * l_p > 64 and many and products(g128, 128) <= 2 * products(g32, 32) else g32


@pytest.mark.parametrize("g_size", [1.0, 1e32])
@pytest.mark.parametrize("shape,qkv,proj,dx_tile", SMHA_TILES)
def test_every_smha_tile(shape, qkv, proj, dx_tile, g_size):
    """Forward and backward of the block with rows that are absent from K segments (out-projection, d_x); a gradient of 1e32 as above."""
    b, m, l_p, d, n, k, c, d_h = shape
    print(f"fp32 smha {shape} gradient {g_size}", flush=True)
    gp, l_a, l = patch_groups(b, l_p, m, c, d), c * l_p, m * l_p
    groups = b * -(-m // gp)
    assert qkv == tile(False, False, b * k, l_a, 3 * d_h)
    assert proj == tile(False, False, groups, gp * l_p, d) and dx_tile == tile(False, True, groups, gp * l_p, d)
    g = torch.Generator(device="cuda").manual_seed(31)
    rnd = lambda *s: torch.randn(s, generator=g, device="cuda")
    x, d_out = rnd(b, l, d), g_size * rnd(b, l, d)
    w = [0.1 * rnd(n, d, d_h) for _ in range(3)] + [0.1 * rnd(n, d_h, d)]
    idx = torch.stack([torch.randperm(n, generator=g, device="cuda")[:k].sort().values for _ in range(b)]).int().contiguous()
    pidx = torch.stack([torch.randperm(m, generator=g, device="cuda")[:c].sort().values for _ in range(b * n)]).int().reshape(b, n, c).contiguous()
    eg, pg = torch.ones((b, n), device="cuda"), torch.ones((b, n, m), device="cuda")
    blk = B.block_desc(b, l, d, n, k, m, c, d_h, B.F32, 0)
    out, dx, dw = torch.empty_like(x), torch.empty_like(x), [torch.empty_like(t) for t in w]
    room = lambda nbytes: torch.empty(nbytes, dtype=torch.uint8, device="cuda")
    B.smha_forward(blk, x, *w, idx, eg, pidx, pg, out, room(B.workspace_bytes(blk, None)))
    B.smha_backward(blk, x, B.smha_weights(None, None, None, *w), idx, eg, pidx, pg, None, d_out, dx, B.smha_weight_grads(*dw),
                    torch.empty_like(eg), torch.empty_like(pg), room(B.smha_backward_workspace_bytes(blk)))
    leaves = [t.double().requires_grad_(True) for t in (x, *w)]
    sample, e = torch.arange(b, device="cuda")[:, None], idx.long()
    tok = (pidx[sample, e].long()[..., None] * l_p + torch.arange(l_p, device="cuda")).reshape(b, k, l_a)
    flat = (sample[..., None] * l + tok).reshape(-1)
    h = leaves[0].reshape(b * l, d)[flat].reshape(b * k, l_a, d)
    q, kk, v = (torch.bmm(h, t[e.reshape(-1)].contiguous()) for t in leaves[1:4])
    o = torch.bmm(torch.softmax(torch.bmm(q, kk.transpose(1, 2).contiguous()) / d_h ** 0.5, -1), v)
    ref = torch.zeros((b * l, d), dtype=torch.float64, device="cuda").index_add(0, flat, torch.bmm(o, leaves[4][e.reshape(-1)].contiguous()).reshape(-1, d))
    grads = torch.autograd.grad((ref * d_out.double().reshape(-1, d)).sum(), leaves)
    for name, y, r in zip(("out", "d_x", "d_wq", "d_wk", "d_wv", "d_wo"), (out, dx, *dw), (ref.detach().reshape(b, l, d), *grads)):
        err = ((y.double() - r).norm() / r.norm()).item()
        print(f"  {name} {err:.2e}", flush=True)
        assert err <= 2e-6   # four contractions and a softmax in a row
