"""The large tiles of the MLP contractions, whose epilogues fetch the residual or Z under the last K-step: rows and columns that end inside a
tile, no residual, with and without the non-temporal accesses.  Against the same products in torch, float32."""
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu

R, GE = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT
SHAPES = {"rows": (2, 8224, 1024), "columns": (2, 8192, 1056)}   # b, l, d: at least 256 tiles of 256 x 256, 32 past the last one
N, K, D_E = 5, 4, 256


def make(b, l, d, flags, D_E=D_E):
    gen = torch.Generator(device="cuda").manual_seed(l + d + flags)
    t = {name: (torch.randn(shape, generator=gen, device="cuda") * std).bfloat16() for name, shape, std in (
        ("u", (b, l, d), 1.0), ("d_out", (b, l, d), 1.0), ("hidden", (b, l, K * D_E), 0.5), ("a_in", (N, d, D_E), 0.03), ("a_out", (N, D_E, d), 0.03))}
    idx = torch.tensor([[0, 1, 3, 4], [0, 2, 3, 4]], dtype=torch.int32, device="cuda")
    gate = torch.softmax(torch.randn(b, N, generator=gen, device="cuda"), 1)
    return B.block_desc(b, l, d, N, K, 1, 1, D_E, B.BF16, flags), t, idx, gate


def close(got, want, what):
    """Two bf16 roundings of intermediates and one of the result, 1.7e-3 each on the average; the worst of 10^7 elements is some 6
    times that of the tensor's rms."""
    got, want = got.float(), want.float()
    err, rms = got - want, want.pow(2).mean().sqrt()
    assert err.norm() / want.norm() <= 6e-3, (what, float(err.norm() / want.norm()))
    assert (err.abs() / torch.maximum(want.abs(), rms)).max() <= 4e-2, what


@pytest.mark.parametrize("once", [False, True])
@pytest.mark.parametrize("flags", [0, R])
@pytest.mark.parametrize("name", list(SHAPES))
def test_down(name, flags, once, monkeypatch):
    monkeypatch.setenv("UOE_STREAM_ONCE_MIN_BYTES", "0" if once else "1e18")
    desc, t, idx, _ = make(*SHAPES[name], flags)
    out = torch.full_like(t["u"], float("nan"))
    B.uome_down(desc, t["hidden"], t["a_out"], t["u"], idx, out)
    torch.cuda.synchronize()
    for s in range(idx.shape[0]):
        want = t["hidden"][s].float() @ t["a_out"][idx[s].long()].reshape(K * D_E, -1).float()
        close(out[s], want + t["u"][s].float() if flags else want, f"sample {s}")


# dH fetches Z: on 256 x 256 tiles with d a multiple of 64; "z_columns": 4 x 288 columns of Z end inside the fifth of them, 32 rows past the last tile too
@pytest.mark.parametrize("once", [False, True])
@pytest.mark.parametrize("name", ["rows", "columns", "z_columns"])
def test_backward(name, once, monkeypatch):
    monkeypatch.setenv("UOE_STREAM_ONCE_MIN_BYTES", "0" if once else "1e18")
    desc, t, idx, gate = make(*SHAPES.get(name, SHAPES["rows"]), R | GE, 288 if name == "z_columns" else D_E)
    grads = [torch.full_like(t[k], float("nan")) for k in ("u", "a_in", "a_out")]
    d_gate = torch.full_like(gate, float("nan"))
    ws = torch.empty(B.uome_backward_workspace_bytes(desc), dtype=torch.uint8, device="cuda")
    B.uome_backward(desc, t["u"], t["a_in"], t["a_out"], idx, gate, None, None, t["d_out"], *grads, d_gate, None, ws)
    torch.cuda.synchronize()
    want_in, want_out, want_gate = torch.zeros_like(t["a_in"], dtype=torch.float32), torch.zeros_like(t["a_out"], dtype=torch.float32), torch.zeros_like(gate)
    for s in range(idx.shape[0]):
        u, g = t["u"][s].float(), t["d_out"][s].float()
        d_u = g.clone()
        for i in idx[s].tolist():
            z, dh, w = u @ t["a_in"][i].float(), g @ t["a_out"][i].float().T, gate[s, i]
            sig = torch.sigmoid(z)
            dz = dh * w * (sig * (1 + z * (1 - sig)))
            want_gate[s, i] = (dh * z * sig).sum()
            d_u += dz @ t["a_in"][i].float().T
            want_in[i] += u.T @ dz
            want_out[i] += (w * z * sig).T @ g
        close(grads[0][s], d_u, "d_u")
    close(grads[1], want_in, "d_a_in")
    close(grads[2], want_out, "d_a_out")
    assert (d_gate - want_gate).norm() / want_gate.norm() <= 6e-3
