"""Values at the ends of what the storage types hold: heads whose v leaves the range of fp16, pre-activations where the
sigmoid is as small as fp32 can hold, gates that are no softmax of anything."""
import numpy as np
import pytest
import torch

import test_gpu_parity as P
from paper_2503_02495_amd import binding as B
from paper_2503_02495_amd import synth

pytestmark = pytest.mark.gpu

R, GE, GP, CA = B.FLAG_RESIDUAL, B.FLAG_GATE_EXPERT, B.FLAG_GATE_PATCH, B.FLAG_CAUSAL
BF = synth.BF16

RANGE = {
    "vr_dh8": P.small(b=2, l=35, d=40, n_a=3, d_h=8, m=5, c=2, k_a=2, n_m=3, d_e=8, k_m=2, dtype=BF),
    "vr_dh40": P.small(b=2, l=84, d=96, n_a=2, d_h=40, m=6, c=3, k_a=1, n_m=2, d_e=32, k_m=1, dtype=BF),
    "vr_dh96": P.small(b=2, l=84, d=64, n_a=2, d_h=96, m=6, c=3, k_a=1, n_m=2, d_e=32, k_m=1, dtype=BF),
    "vr_d72": P.small(b=2, l=192, d=72, n_a=3, d_h=64, m=6, c=4, k_a=2, n_m=2, d_e=32, k_m=1, dtype=BF),
}


@pytest.mark.parametrize("name", list(RANGE))
@pytest.mark.parametrize("power", [20, -24])
def test_smha_range_of_v(name, power, monkeypatch):
    """bf16 blocks off the 32-multiples: v and its probabilities are held in bf16 and fp32, so v may have any magnitude
    bf16 holds (2^20 here: past fp16's 65504; 2^-24: below its smallest value).  A power of two on W^v scales the exact
    result by itself: same bound as unscaled."""
    plain = synth.make_inputs

    def scaled(cfg, **kw):
        inp = plain(cfg, **kw)
        inp.wv = inp.wv * np.float32(2.0 ** power)
        return inp

    monkeypatch.setitem(P.EDGE_CONFIGS, name, RANGE[name])
    monkeypatch.setattr(synth, "make_inputs", scaled)
    print(f"range of v {name} 2^{power}", flush=True)
    P.run_smha_stage(name, 0)
    P.run_smha_variant(name, CA, 8, 0.2)


# bf16 values at which exp(-z) is between 2^126 and the largest fp32: its reciprocal is no normal number, z times it is
TAIL = [-88.5, -88.0, -87.5]


def silu64(z):
    return z / (1.0 + np.exp(-z))


def one_hot(shape, at, value):
    t = torch.zeros(shape, dtype=torch.bfloat16, device="cuda")
    t[at] = value
    return t


@pytest.mark.parametrize("select", [False, True])
def test_silu_tail_off_32(select):
    """The MLP's activation where widths are no multiple of 32: division and exponential in fp32, rounded once, for
    pre-activations down to -88 (relative error of a bf16 result: 2^-9, bound 2^-8)."""
    z = np.array(TAIL + [-60.0, -1.5, 0.5, 30.0])
    l, d, d_e = len(z), 72, 40
    u = torch.zeros((1, l, d), dtype=torch.bfloat16, device="cuda")
    u[0, :, 0] = torch.tensor(z, dtype=torch.float32).to(torch.bfloat16).cuda()
    a_in = one_hot((1, d, d_e), (0, 0), 1.0)
    idx = torch.zeros((1, 1), dtype=torch.int32, device="cuda")
    if not select:
        blk = B.block_desc(1, l, d, 1, 1, 1, 1, d_e, B.BF16, 0)
        hidden = torch.empty((1, l, d_e), dtype=torch.bfloat16, device="cuda")
        B.uome_up(blk, u, a_in, idx, None, hidden)
        got = hidden[0].float().cpu().numpy()
    else:   # out = hidden A^O with a single one in A^O: the first hidden column
        blk = B.block_desc(1, l, d, 1, 1, l, l - 1, d_e, B.BF16, 0)
        pidx = torch.arange(l - 1, dtype=torch.int32, device="cuda").reshape(1, 1, l - 1)
        out = torch.empty_like(u)
        ws = torch.empty(B.workspace_bytes(None, blk), dtype=torch.uint8, device="cuda")
        B.uome_forward(blk, u, a_in, one_hot((1, d_e, d), (0, 0, 0), 1.0), idx, None, pidx, None, out, ws)
        got = out[0, :-1, :1].float().cpu().numpy()
        z = z[:-1]
    want = silu64(z)[:, None]
    assert np.all(np.abs(got - want) <= 2.0 ** -8 * np.abs(want)), (got[:, 0], want[:, 0])


@pytest.mark.parametrize("z", TAIL)
@pytest.mark.parametrize("b,l,d,d_e,m", [(1, 32, 32, 32, 1), (24, 2048, 32, 256, 1), (1, 64, 32, 32, 2), (1, 20, 24, 8, 1)],
                         ids=["one_launch", "two_launches", "data_selection", "any_shape"])
def test_uome_backward_sigmoid_tail(b, l, d, d_e, m, z):
    """dL/d(gate) = sum dH SiLU(Z) is an fp32 output: pre-activations of -88 must count with their own value (fp32
    exponential of 88: 88 * 2^-24 = 5e-6 relative; bound 1e-4)."""
    print(f"sigmoid tail b={b} l={l} d={d} d_e={d_e} m={m} z={z}", flush=True)
    c = m // 2 if m > 1 else 1
    blk = B.block_desc(b, l, d, 1, 1, m, c, d_e, B.BF16, GE)
    u, a_in = one_hot((b, l, d), (slice(None), slice(None), 0), z), one_hot((1, d, d_e), (0, 0), 1.0)
    a_out, d_out = one_hot((1, d_e, d), (0, slice(None), 0), 1.0), one_hot((b, l, d), (slice(None), slice(None), 0), 2.0 ** 40)
    idx, gate = torch.zeros((b, 1), dtype=torch.int32, device="cuda"), torch.ones((b, 1), device="cuda")
    pidx = torch.zeros((b, 1, c), dtype=torch.int32, device="cuda") if m > 1 else None
    d_u, d_gate = torch.empty_like(u), torch.empty_like(gate)
    ws = torch.empty(B.uome_backward_workspace_bytes(blk), dtype=torch.uint8, device="cuda")
    B.uome_backward(blk, u, a_in, a_out, idx, gate, pidx, None, d_out, d_u, torch.empty_like(a_in), torch.empty_like(a_out),
                    d_gate, None, ws)
    got = d_gate.double().cpu().numpy()
    want = (l // m) * c * d_e * 2.0 ** 40 * silu64(z)
    assert np.all(np.abs(got - want) <= 1e-4 * abs(want)), (got.ravel()[:2], want)


@pytest.mark.parametrize("b,l", [(128, 32), (24, 2048)], ids=["one_launch", "two_launches"])
def test_uome_backward_sigmoid_over_its_range(b, l):
    """z sigmoid(z) of up to 4096 pre-activations from -88 to 88 (the fp32 exponential ends at 88.7), alone in d_gate.  Two fp32 roundings of the exponential's argument, |z| 2^-24 each,
    and some eight of one ulp and less behind them; below 2^-126 the steps of fp32's smallest numbers.  NaN
    comes out as NaN."""
    n, d = 32, 32
    step, top = torch.arange(b, dtype=torch.float32) * (128 // b), torch.tensor([88.0 * 0.75 ** i for i in range(16)])
    u = torch.zeros((b, l, d), dtype=torch.bfloat16, device="cuda")
    u[:, 0, 0] = (1.0 - step / 256).to(torch.bfloat16).cuda()                   # 1/256 steps down to 0.5: exact
    a_in = torch.zeros((n, d, 32), dtype=torch.bfloat16, device="cuda")
    a_in[:, 0, 0] = torch.cat([top, -top]).to(torch.bfloat16).cuda()
    z = (u[:, :1, 0].double() * a_in[None, :, 0, 0].double()).to(torch.bfloat16 if l > 32 else torch.float32).double().cpu().numpy()   # Z is stored in bf16 between two launches
    blk = B.block_desc(b, l, d, n, n, 1, 1, 32, B.BF16, GE)
    a_out, d_out = one_hot((n, 32, d), (slice(None), 0, 0), 1.0), one_hot((b, l, d), (slice(None), 0, 0), 2.0 ** 40)
    idx = torch.arange(n, dtype=torch.int32, device="cuda").repeat(b, 1)
    gate = torch.ones((b, n), device="cuda")
    d_gate, ws = torch.empty_like(gate), torch.empty(B.uome_backward_workspace_bytes(blk), dtype=torch.uint8, device="cuda")
    run = lambda: B.uome_backward(blk, u, a_in, a_out, idx, gate, None, None, d_out, torch.empty_like(u), torch.empty_like(a_in), torch.empty_like(a_out), d_gate, None, ws)
    run()
    got, want = d_gate.double().cpu().numpy() * 2.0 ** -40, silu64(z)
    off = np.abs(got - want) - np.abs(want) * (2 * np.abs(z) + 16) * 2.0 ** -24 - np.abs(z) * 2.0 ** -149
    assert off.max() <= 0, (z.ravel()[off.argmax()], got.ravel()[off.argmax()], want.ravel()[off.argmax()])
    a_in[0, 0, 0] = float("nan")
    run()
    again = d_gate.double().cpu().numpy() * 2.0 ** -40
    assert np.all(np.isnan(again[:, 0])) and np.array_equal(again[:, 1:], got[:, 1:])


@pytest.mark.parametrize("name", ["tiny", "bf16_noise", "bf16_n32"])
def test_route_backward_any_gates(name):
    """The formula of uoe_route_backward holds for whatever gates a caller hands over, not only for rows that sum to one."""
    cfg = P.get_cfg(name)
    print(f"route backward, gates that do not sum to one: {name}", flush=True)
    inp = synth.make_inputs(cfg, w_std=0.06)
    rng = np.random.default_rng(3)
    ge = rng.uniform(0.1, 1.0, (cfg.b, cfg.n_a)).astype(np.float32)
    gp = rng.uniform(0.1, 1.0, (cfg.b, cfg.n_a, cfg.m)).astype(np.float32)
    d_ge, d_gp = synth.make_gate_grads(cfg, cfg.n_a, cfg.m)
    d_x0 = synth.make_upstream_grad(cfg)
    dev = P.DeviceLayer(inp, R, R)
    f32 = lambda a: P.to_device(a, synth.F32, dev.device)
    d_x = P.to_device(d_x0, cfg.dtype, dev.device)
    d_we, d_wb, d_wa = (torch.empty_like(t) for t in (dev.a_w_expert, dev.a_w_b, dev.a_w_a))
    ws = torch.empty(B.route_backward_workspace_bytes(dev.smha), dtype=torch.uint8, device=dev.device)
    B.route_backward(dev.smha, dev.x, dev.a_w_expert, dev.a_w_b, dev.a_w_a, f32(ge), f32(gp), f32(d_ge), f32(d_gp),
                     d_x, d_we, d_wb, d_wa, ws)
    torch.cuda.synchronize()
    want = P.oracle.route_backward(inp.x, inp.a_w_expert, inp.a_w_b, inp.a_w_a, ge, gp, d_ge, d_gp)
    errs = {"d_x": P.scaled_err(P.to_host(d_x), d_x0.astype(np.float64) + want.d_x),
            "d_w_expert": P.grad_err(P.to_host(d_we), want.d_w_expert),
            "d_w_b": P.grad_err(P.to_host(d_wb).T, want.d_w_b.T), "d_w_a": P.grad_err(P.to_host(d_wa).T, want.d_w_a.T)}
    print(" ".join(f"{k} {v:.3e}" for k, v in errs.items()), flush=True)
    assert max(errs.values()) <= P.TOL[cfg.dtype], errs


@pytest.mark.parametrize("flags", [0, R | GE | GP | CA])
def test_smha_backward_equal_keys_large_logits(flags):
    """fp32: every key of a unit is the same, with logits around 200.  The probabilities are then 1 / (number of keys) to the
    last bit, whatever the logits are; a softmax held as a log-sum-exp of 300 is off by 2^-16.  d_wv and d_wo take the
    probabilities times sums of at most 120 terms: 2e-6 (sqrt(120) * 2^-24 = 7e-7)."""
    cfg = P.small(b=2, l=60, d=40, n_a=2, d_h=24, m=6, c=5, k_a=1, n_m=2, d_e=8, k_m=1)
    print(f"equal keys, large logits, flags={flags}", flush=True)
    inp = synth.make_inputs(cfg, w_std=0.1)
    inp.x[:] = inp.x[:, :1]
    q = np.einsum("bd,ndh->bnh", inp.x[:, 0], inp.wq)
    inp.wq = inp.wk = (inp.wq * np.sqrt(200.0 * np.sqrt(cfg.d_h) / np.mean(np.sum(q * q, -1)))).astype(np.float32)
    d_out = synth.make_upstream_grad(cfg)
    dev = P.DeviceLayer(inp, flags, R)
    ref = P.oracle.route(inp.x, cfg.n_a, cfg.k_a, cfg.m, cfg.c, inp.a_w_expert, inp.a_w_b, inp.a_w_a, None, None)
    ge, gp = ref.expert_gate.astype(np.float32), ref.patch_gate.astype(np.float32)
    i32, f32 = (lambda a: torch.from_numpy(a).to(dev.device)), (lambda a: P.to_device(a, synth.F32, dev.device))
    got = dev.smha_backward(f32(d_out), i32(ref.expert_id), f32(ge), i32(ref.patch_id), f32(gp))
    want = P.oracle.smha_backward(inp.x, inp.wq, inp.wk, inp.wv, inp.wo, ref.expert_id, ge, ref.patch_id, gp, cfg.m, d_out, flags)
    errs = {"d_wv": P.fro_err(P.to_host(got[3]), want.d_wv), "d_wo": P.fro_err(P.to_host(got[4]), want.d_wo)}
    print(errs, flush=True)
    assert max(errs.values()) <= 2e-6, errs
