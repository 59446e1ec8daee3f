"""The SMHA block's backward pass off the 32-grid with as many units as it takes (b * k up to 65535), gate gradients among its results, against
the same samples in calls of 4096 units: what a sample gets depends on that sample only, up to the order of fp32 sums (contractions
choose their tiles by the size of the call: 1e-5 of the largest value, over sums of at most 40 products)."""
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu

R, GE, GP = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT, B.FLAG_GATE_PATCH


def backward(t, first, last, n, k, width):
    x, b, l, d = t["x"][first:last], last - first, t["x"].shape[1], t["x"].shape[2]
    desc = B.block_desc(b, l, d, n, k, 1, 1, width, B.F32, R | GE | GP)
    nan = lambda *s: torch.full(s, float("nan"), device="cuda")
    d_x, d_ge, d_gp = nan(b, l, d), nan(b, n), nan(b, n, 1)
    dw = [nan(n, d, width) for _ in range(3)] + [nan(n, width, d)]
    ws = torch.empty(B.smha_backward_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    w = B.smha_weights(None, None, None, t["wq"], t["wk"], t["wv"], t["wo"])
    B.smha_backward(desc, x, w, t["idx"][first:last], t["ge"][first:last], t["pidx"][first:last], t["gp"][first:last], None, t["d_out"][first:last], d_x,
                    B.smha_weight_grads(*dw), d_ge, d_gp, ws)
    torch.cuda.synchronize()
    return d_x, d_ge, d_gp, dw


@pytest.mark.parametrize("b,k,n,l", [(65535, 1, 2, 8), (21845, 3, 4, 40)], ids=["one_block_of_rows", "two"])
def test_units_up_to_the_bound(b, k, n, l):
    print(f"smha backward of {b} samples, {k} of {n} experts, {l} tokens", flush=True)
    d, width, gen = 8, 8, torch.Generator(device="cuda").manual_seed(l)
    draw = lambda *s: torch.randn(s, generator=gen, device="cuda")
    t = {"x": draw(b, l, d), "d_out": draw(b, l, d), **{w: 0.2 * draw(n, d, width) for w in ("wq", "wk", "wv")}, "wo": 0.2 * draw(n, width, d),
         "ge": torch.rand(b, n, generator=gen, device="cuda"), "gp": torch.rand(b, n, 1, generator=gen, device="cuda"),
         "idx": torch.argsort(torch.rand(b, n, generator=gen, device="cuda"), 1)[:, :k].sort(1)[0].to(torch.int32).contiguous(),
         "pidx": torch.zeros(b, n, 1, device="cuda", dtype=torch.int32)}
    *whole, dw = backward(t, 0, b, n, k, width)
    step, sums = 4096 // k, [torch.zeros_like(w, dtype=torch.float64) for w in dw]
    for first in range(0, b, step):
        last = min(first + step, b)
        *some, part = backward(t, first, last, n, k, width)
        for got, want in zip(whole, some):
            assert torch.isfinite(got[first:last]).all()
            assert (got[first:last] - want).abs().max() <= 1e-5 * want.abs().max(), first
        for s, w in zip(sums, part):
            s += w
    for got, want in zip(dw, sums):
        assert (got - want).abs().max() <= 1e-5 * want.abs().max()
