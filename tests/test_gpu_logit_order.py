"""The order in which the chunks' partial expert logits are added, which decides the last bits of the gates and so those of every gradient behind
them: chunks equal modulo 512 / n one after the other, then groups equal modulo 16, then 16 lanes by halves.  Each chunk's partial is one
number, exact, and pairs of 2^24 that cancel only in part of the orders move a logit by whole units if the order is another."""
import numpy as np
import pytest
import torch

from paper_2503_02495_amd import binding as B

pytestmark = pytest.mark.gpu

CASES = [  # n, chunks, bf16
    (2, 300, True), (3, 512, True), (4, 700, True), (7, 511, True), (8, 130, True), (8, 512, True), (9, 1000, True), (15, 13, True), (16, 700, True),
    (17, 1023, True), (31, 600, True), (32, 512, True), (5, 700, False), (12, 333, False), (32, 900, False),
]


def logits(p, n):
    groups = 512 // n
    s, t = np.zeros((n, groups), np.float32), np.zeros((n, 16), np.float32)
    for c in range(p.shape[1]):
        s[:, c % groups] += p[:, c]
    for g in range(groups):
        t[:, g % 16] += s[:, g]
    for off in (1, 2, 4, 8):
        t = t + t[:, np.arange(16) ^ off]
    return t[:, 0]


@pytest.mark.parametrize("n,chunks,bf16", CASES)
def test_order_of_the_sums(n, chunks, bf16):
    rng = np.random.default_rng(n * 1024 + chunks)
    b, tokens = (2, 1) if bf16 else (1, 4)   # tokens of a chunk: bf16 below 1024 a sample, fp32 below 4096 in all
    l, d = chunks * tokens, 8
    p = rng.integers(-16, 17, (n, chunks)).astype(np.float32) / 8
    for e in range(n):
        at = rng.permutation(chunks)[:chunks // 4 * 2]
        p[e, at[0::2]], p[e, at[1::2]] = 2.0 ** 24, -2.0 ** 24
    w = np.zeros((n, l, d), np.float32)
    w[:, ::tokens, 0] = p
    x = np.stack([np.ones((l, d)), np.full((l, d), 0.5)])[:b].astype(np.float32)
    dt = torch.bfloat16 if bf16 else torch.float32
    gate = torch.full((b, n), float("nan"), device="cuda")
    idx = torch.full((b, 1), -1, dtype=torch.int32, device="cuda")
    desc = B.block_desc(b, l, d, n, 1, 1, 1, 8, B.BF16 if bf16 else B.F32, 0)
    ws = torch.empty(B.workspace_bytes(None, desc), dtype=torch.uint8, device="cuda")
    B.route(desc, torch.from_numpy(x).to(dt).cuda(), torch.from_numpy(w.reshape(n, l * d)).to(dt).cuda(), None, None, None, None, idx, gate, None, None, ws)
    torch.cuda.synchronize()
    z = np.stack([logits(p, n), logits(p * 0.5, n)])[:b].astype(np.float64)
    want = np.exp(z - z.max(1, keepdims=True))
    want /= want.sum(1, keepdims=True)
    got = gate.cpu().numpy().astype(np.float64)
    # the logits are exact; exp of a difference of at most 100 (rounded: 2^-18 of it), the sum and the quotient in fp32
    shown = z - z.max(1, keepdims=True) > -80
    assert (np.abs(got - want)[shown] <= 1e-5 * want[shown] + 1e-30).all()
    assert (idx.cpu().numpy()[:, 0] == z.argmax(1)).all()
