"""The bf16 attention kernel that gives every head two waves (half the keys of
each tile each), and the calls without a mask tensor, whose rows and live lists
the kernels compute from coordinates.

Against the float64 oracle with the bars of the other parity tests: bf16
operands and weights give errors near 2^-9 of the values, max-abs 1e-2 and
mean-abs 1e-3 for N(0,1) inputs.
"""
import numpy as np
import pytest
import torch

import oracle
from workloads import random_block_mask, small_qkv

pytestmark = pytest.mark.gpu


def steel():
    import paper_2607_09385_amd as s
    return s


def check(got, want, what):
    err = np.abs(got.double().cpu().numpy() - want)
    assert np.isfinite(err).all(), what
    assert err.max() <= 1e-2, f"{what}: max abs error {err.max()}"
    assert err.mean() <= 1e-3, f"{what}: mean abs error {err.mean()}"


CASES = [
    # B, Hq, Hkv, S_q, S_k, D, causal, masked
    (1, 1, 1, 1, 1, 64, True, False),
    (1, 2, 2, 1, 63, 128, True, False),
    (1, 2, 1, 33, 65, 64, False, False),
    # live lists around the 64 entries a wave holds, aligned and ragged
    (1, 1, 1, 64, 64 * 64, 64, False, False),
    (1, 2, 1, 70, 65 * 64, 128, True, False),
    (1, 4, 1, 20, 129 * 64 + 5, 128, False, False),
    (1, 3, 3, 130, 66 * 64 - 1, 64, True, True),
    # packs of 4 at D = 128 around the 256 up to which two heads share a workgroup
    (16, 16, 4, 256, 256, 128, True, False),
    (13, 16, 4, 300, 300, 128, True, False),
    # dead query rows, heads and packs not a multiple of 8
    (1, 3, 3, 300, 90, 64, True, False),
    (3, 12, 3, 200, 330, 128, True, True),
    (2, 10, 5, 191, 257, 64, True, True),
]


@pytest.mark.parametrize("case", CASES, ids=lambda c: "x".join(str(int(v)) for v in c))
def test_against_oracle(case):
    B, Hq, Hkv, S_q, S_k, D, causal, masked = case
    q, k, v = small_qkv(11, B, Hq, Hkv, S_q, S_k, D)
    nQB, nKB = -(-S_q // 64), -(-S_k // 64)
    m = random_block_mask(np.random.default_rng(5), B, Hq, nQB, nKB, p=0.6) if masked else None
    out = torch.full((B, Hq, S_q, D), float("nan"), dtype=torch.float32, device="cuda")
    steel().attn_fwd(q.cuda(), k.cuda(), v.cuda(), None if m is None else torch.from_numpy(m).cuda(),
                     scale=D ** -0.5, causal=causal, out=out)
    check(out, oracle.attention(q, k, v, m, D ** -0.5, causal, 64), str(case))


@pytest.mark.parametrize("D,Hq,Hkv", [(64, 2, 2), (128, 2, 2), (64, 8, 2), (128, 8, 2)])
def test_growing_maxima(D, Hq, Hkv):
    """Scores that grow along the keys move every row's running maximum by far
    more than the deferred rescale allows (2^24), several times per row."""
    S = 512
    q, k, v = small_qkv(3, 1, Hq, Hkv, S, S, D)
    grow = (1.0 + 40.0 * torch.arange(S) / S)[None, None, :, None]
    k = (k.float() * grow).to(torch.bfloat16)
    out = steel().attn_fwd(q.cuda(), k.cuda(), v.cuda(), scale=D ** -0.5, causal=False)
    # scores up to ~150: their bf16-operand fp32 sums are exact to ~2e-5, the
    # weights to 2^-9 as everywhere
    check(out, oracle.attention(q, k, v, None, D ** -0.5, False, 64), f"D={D}")


@pytest.mark.parametrize("shape", [
    # B, Hq, Hkv, S_q, S_k, D, causal, window, sink
    (1, 8, 8, 512, 512, 64, True, 2, 1),
    (1, 3, 3, 513, 700, 64, True, 3, 0),
    (2, 8, 2, 700, 513, 128, False, 1, 2),
    (1, 12, 3, 1000, 1000, 64, True, 5, 100),
    (1, 4, 2, 320, 1280, 128, True, 1000, 0),
    (9, 16, 4, 640, 640, 128, True, 2, 1),
    (1, 2, 2, 900, 100, 128, True, 2, 1),
], ids=lambda c: "x".join(str(int(v)) for v in c))
def test_coordinates_equal_mask_tensor(shape):
    B, Hq, Hkv, S_q, S_k, D, causal, win, sink = shape
    q, k, v = (t.cuda() for t in small_qkv(7, B, Hq, Hkv, S_q, S_k, D))
    nQB, nKB = -(-S_q // 64), -(-S_k // 64)
    i, j = np.arange(nQB)[:, None], np.arange(nKB)[None, :]
    m = ((j <= i) & (j > i - win)) | (j < sink)
    m = torch.from_numpy(np.broadcast_to(m, (B, Hq, nQB, nKB)).astype(np.uint8).copy()).cuda()
    s = steel()
    assert torch.equal(s.attn_fwd_window(q, k, v, win, sink, causal=causal),
                       s.attn_fwd(q, k, v, m, causal=causal))
    assert torch.equal(s.attn_fwd(q, k, v, None, causal=causal),
                       s.attn_fwd(q, k, v, torch.ones_like(m), causal=causal))
    for fp8 in ("pv", "all"):
        a = s.attn_fwd_lse(q, k, v, None, causal=causal, causal_offset=37, fp8=fp8)
        b = s.attn_fwd_lse(q, k, v, torch.ones_like(m), causal=causal, causal_offset=37, fp8=fp8)
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1])
