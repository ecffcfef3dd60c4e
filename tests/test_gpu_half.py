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
    more than the deferred rescale allows (2^8), several times per row."""
    S = 512
    q, k, v = small_qkv(3, 1, Hq, Hkv, S, S, D)
    grow = (1.0 + 40.0 * torch.arange(S) / S)[None, None, :, None]
    k = (k.float() * grow).to(torch.bfloat16)
    out = steel().attn_fwd(q.cuda(), k.cuda(), v.cuda(), scale=D ** -0.5, causal=False)
    # scores up to ~150: their bf16-operand fp32 sums are exact to ~2e-5, the
    # weights to 2^-9 as everywhere
    check(out, oracle.attention(q, k, v, None, D ** -0.5, False, 64), f"D={D}")


@pytest.mark.parametrize("half", [0, 1])
@pytest.mark.parametrize("D", [64, 128])
def test_growing_maxima_of_one_half(D, half):
    """Only 32 of a block's 64 rows have growing maxima; the others' stay."""
    S = 512
    q, k, v = small_qkv(4, 1, 1, 1, S, S, D)
    grow = (1.0 + 40.0 * torch.arange(S) / S)[None, None, :, None]
    still = (torch.arange(S) // 32 % 2 != half)[None, None, :, None]
    q = torch.where(still, q.float() / 64, q.float()).to(torch.bfloat16)
    k = (k.float() * grow).to(torch.bfloat16)
    out = steel().attn_fwd(q.cuda(), k.cuda(), v.cuda(), scale=D ** -0.5, causal=False)
    check(out, oracle.attention(q, k, v, None, D ** -0.5, False, 64), f"D={D}")


@pytest.mark.parametrize("shape", [
    # B, Hq, Hkv, S_q, S_k, D, causal, window, sink
    (1, 8, 8, 512, 512, 64, True, 2, 1),
    (1, 3, 3, 513, 700, 64, True, 3, 0),
    (2, 8, 2, 700, 513, 128, False, 1, 2),
    (1, 12, 3, 950, 950, 64, True, 5, 100),
    (1, 4, 2, 320, 900, 128, True, 1000, 0),
    (9, 16, 4, 640, 640, 128, True, 2, 1),
    (1, 2, 2, 900, 100, 128, True, 2, 1),
    # many heads: several ranges of them, the last a smaller one; contiguous
    # shares of a window over heads that are no multiple of 8
    (9, 17, 17, 960, 960, 64, False, 3, 1),
    (3, 50, 50, 900, 960, 128, True, 2, 1),
    (20, 32, 8, 900, 960, 64, False, 3, 1),
    # groups of several units: dealt to the XCDs by group, eight and more of them
    (2, 40, 8, 300, 400, 64, False, 3, 1),
    (3, 28, 4, 300, 400, 128, True, 2, 1),
    (2, 64, 8, 200, 400, 128, True, 2, 0),
    # few query blocks of nearly equal lists: ranges bounded by keys and values,
    # and 64-row waves where 128 workgroups per XCD have lists of one length
    (80, 8, 8, 130, 900, 64, True, 2, 0),
    (32, 8, 8, 256, 1100, 128, True, 2, 0),
], ids=lambda c: "x".join(str(int(v)) for v in c))
def test_coordinates_equal_mask_tensor(shape):
    """Bit for bit where the lists are not split (fewer than 16 key blocks)."""
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


SPLIT = [
    # B, Hq, Hkv, S_q, S_k, D, causal: few query blocks, long key lists
    (1, 4, 1, 1, 2048, 128, True),
    (3, 8, 2, 1, 1111, 64, True),
    (2, 8, 1, 8, 1024, 128, True),     # 8 heads x 8 rows fill a tile
    (1, 8, 1, 9, 1500, 64, False),     # 4 heads x 9 rows
    (1, 6, 2, 21, 1024, 128, True),    # 3 heads x 21 rows
    (1, 5, 5, 64, 2000, 64, True),     # one head per tile
    (1, 8, 4, 65, 1090, 128, True),    # two query blocks, packs of 2
    (1, 4, 1, 200, 3000, 128, True),
    (1, 2, 2, 300, 1024, 64, False),
    (1, 1, 1, 1100, 1030, 128, True),  # dead rows at the start
    (8, 40, 8, 13, 1024, 64, True),    # 320 units of one head, 5 per group
]


@pytest.mark.parametrize("case", SPLIT, ids=lambda c: "x".join(str(int(v)) for v in c))
def test_split_lists(case):
    """Lists cut into segments and several heads in one tile's rows: output
    and log-sum-exp against the oracle, and the other forms of the call, which
    split alike, bit for bit."""
    B, Hq, Hkv, S_q, S_k, D, causal = case
    q, k, v = small_qkv(13, B, Hq, Hkv, S_q, S_k, D)
    qc, kc, vc = q.cuda(), k.cuda(), v.cuda()
    want, want_lse = oracle.attention_lse(q, k, v, None, D ** -0.5, causal, 64, S_k - S_q)
    s = steel()
    out = torch.full((B, Hq, S_q, D), float("nan"), dtype=torch.float32, device="cuda")
    lse = torch.full((B, Hq, S_q), float("nan"), dtype=torch.float32, device="cuda")
    s.attn_fwd_lse(qc, kc, vc, scale=D ** -0.5, causal=causal, out=out, lse=lse)
    check(out, want, str(case))
    got = lse.double().cpu().numpy()
    dead = np.isneginf(want_lse)
    assert np.array_equal(np.isneginf(got), dead)
    assert np.abs(got[~dead] - want_lse[~dead]).max(initial=0.0) <= 1e-3
    assert torch.equal(out, s.attn_fwd(qc, kc, vc, scale=D ** -0.5, causal=causal))
    bf, _ = s.attn_fwd_lse(qc, kc, vc, scale=D ** -0.5, causal=causal, out_dtype=torch.bfloat16)
    assert torch.equal(bf, out.to(torch.bfloat16))
    other = torch.full_like(out, float("nan"))
    st = s._lib.load().steel_attn_fwd_noalloc(
        qc.data_ptr(), kc.data_ptr(), vc.data_ptr(), None, other.data_ptr(), B, Hq, Hkv, S_q, S_k,
        D, 64, D ** -0.5, int(causal), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert torch.equal(out, other)


def test_split_window():
    q, k, v = (t.cuda() for t in small_qkv(17, 1, 4, 1, 640, 8192, 64))
    qb, kb = np.arange(10)[:, None], np.arange(128)[None, :]
    m = (((kb <= qb) & (kb > qb - 2)) | (kb < 70)).astype(np.uint8)
    m = np.ascontiguousarray(np.broadcast_to(m, (1, 4, 10, 128)))
    got = steel().attn_fwd_window(q, k, v, 2, 70, causal=False)
    check(got, oracle.attention(q.cpu(), k.cpu(), v.cpu(), m, 64 ** -0.5, False, 64), "window")


@pytest.mark.parametrize("B,Hq,Hkv,S_q,S_k,D,uniform", [
    # masks whose packs are all uniform, some, or none, heads over the 8 XCDs
    # evenly and not, rows of one and of several 256-block reads (S_k > 16384),
    # packs beyond one sort round (1024), live counts beyond 128
    (1, 8, 8, 700, 700, 64, 0.0),
    (1, 36, 9, 500, 500, 128, 0.5),
    (2, 32, 8, 4200, 300, 64, 1.0),
    (1, 4, 1, 130, 16500, 64, 0.5),
    (1, 16, 8, 2100, 2100, 64, 0.97),
], ids=str)
def test_index_of_mask_tensors(B, Hq, Hkv, S_q, S_k, D, uniform):
    """Every row is dealt out exactly once, whichever list it is in: outputs
    against the oracle in a buffer of NaN."""
    rng = np.random.default_rng(B * 100 + Hq)
    nQB, nKB = -(-S_q // 64), -(-S_k // 64)
    m = random_block_mask(rng, B, Hq, nQB, nKB, p=0.7)
    G = Hq // Hkv
    shared = rng.random((B, Hkv, nQB)) < uniform  # these groups share one live set
    for b, g, qb in np.argwhere(shared):
        m[b, g * G:(g + 1) * G, qb] = m[b, g * G, qb]
    q, k, v = small_qkv(19, B, Hq, Hkv, S_q, S_k, D)
    out = torch.full((B, Hq, S_q, D), float("nan"), dtype=torch.float32, device="cuda")
    steel().attn_fwd(q.cuda(), k.cuda(), v.cuda(), torch.from_numpy(m).cuda(), causal=False, out=out)
    assert torch.isfinite(out).all()
    rows = np.unique(np.concatenate([[0, S_q - 1], rng.integers(0, S_q, 200)]))
    blocks = np.unique(rows // 64)[:6]
    for b in range(B):
        for qb in blocks:
            r0, r1 = qb * 64, min(qb * 64 + 64, S_q)
            want = oracle.attention(q[b:b + 1, :, r0:r1], k[b:b + 1], v[b:b + 1],
                                    np.ascontiguousarray(m[b:b + 1, :, qb:qb + 1]), D ** -0.5, False, 64)
            check(out[b:b + 1, :, r0:r1], want, f"batch {b} block {qb}")


@pytest.mark.parametrize("D,Hq,Hkv,S_q,S_k,causal", [
    (64, 3, 3, 130, 450, False), (64, 3, 3, 448, 448, True), (128, 3, 3, 130, 450, False),
    (128, 3, 3, 448, 448, True), (64, 4, 2, 448, 450, True), (128, 4, 2, 448, 450, True),
    (128, 2, 2, 900, 900, True),
], ids=str)
def test_waves_of_32_rows_equal_waves_of_64(D, Hq, Hkv, S_q, S_k, causal):
    """One problem by itself (few workgroups: 32 query rows per wave) and as
    part of a large batch (64): the same rows bit for bit, with an index and
    without, a block's maxima growing in one half only."""
    B = 1 + 8 * 900 // (Hkv * -(-S_q // 64))
    q, k, v = small_qkv(23, 1, Hq, Hkv, S_q, S_k, D)
    grow = (1.0 + 20.0 * torch.arange(S_k) / S_k)[None, None, :, None]
    still = (torch.arange(S_q) // 32 % 2 == 0)[None, None, :, None]
    q = torch.where(still, q.float() / 64, q.float()).to(torch.bfloat16).cuda()
    k, v = (k.float() * grow).to(torch.bfloat16).cuda(), v.cuda()
    many = [t.expand(B, -1, -1, -1).contiguous() for t in (q, k, v)]
    mask = lambda b: torch.ones((b, Hq, -(-S_q // 64), -(-S_k // 64)), dtype=torch.uint8, device="cuda")
    s = steel()
    for with_index in (False, True):
        one = s.attn_fwd(q, k, v, mask(1) if with_index else None, causal=causal)
        all_ = s.attn_fwd(*many, mask(B) if with_index else None, causal=causal)
        assert torch.equal(one.expand_as(all_), all_)
    check(one, oracle.attention(q.cpu(), k.cpu(), v.cpu(), None, D ** -0.5, causal, 64), "one problem")


def forms(q, k, v, causal):
    """One problem without a mask tensor, in every form that takes none, and
    as a mask tensor and plans."""
    B, Hq, S_q, D = q.shape
    Hkv, S_k = k.shape[1:3]
    nQB, nKB = -(-S_q // 64), -(-S_k // 64)
    s = steel()
    other = torch.full((B, Hq, S_q, D), float("nan"), dtype=torch.float32, device="cuda")
    st = s._lib.load().steel_attn_fwd_noalloc(
        q.data_ptr(), k.data_ptr(), v.data_ptr(), None, other.data_ptr(), B, Hq, Hkv, S_q, S_k, D, 64,
        D ** -0.5, int(causal), torch.cuda.current_stream().cuda_stream)
    assert st == 0
    ones = torch.ones((B, Hq, nQB, nKB), dtype=torch.uint8, device="cuda")
    plain = {"fwd": s.attn_fwd(q, k, v, causal=causal),
             "lse": s.attn_fwd_lse(q, k, v, causal=causal)[0],
             "window": s.attn_fwd_window(q, k, v, nQB + nKB, nKB, causal=causal),
             "noalloc": other}
    indexed = {"mask": s.attn_fwd(q, k, v, ones, causal=causal),
               "plan": s.Plan(None, B, Hq, Hkv, S_q, S_k, causal=causal).run(q, k, v),
               "plan of mask": s.Plan(ones, B, Hq, Hkv, S_q, S_k, causal=causal).run(q, k, v)}
    return plain, indexed


@pytest.mark.parametrize("B,Hq,Hkv,S_q,S_k,D,causal,same", [
    # one query block: a head per key/value head, and several (shared tiles), with
    # packs of 4 at D = 128 beyond the 256 up to which two heads share a workgroup
    (33, 8, 8, 1, 300, 64, True, True),
    (5, 3, 3, 64, 900, 128, False, True),
    (33, 32, 8, 1, 300, 128, True, False),
    (3, 16, 8, 20, 900, 64, False, False),
    (2, 6, 2, 21, 640, 128, True, False),
    (2, 10, 2, 13, 700, 64, True, False),
    # several query blocks, whole and split lists
    (2, 8, 2, 65, 900, 128, True, True),
    (1, 8, 2, 100, 3000, 64, True, False),
    (70, 8, 1, 1, 2000, 128, True, False),
], ids=str)
def test_forms_agree(B, Hq, Hkv, S_q, S_k, D, causal, same):
    """Without a mask tensor every call gives the same bits, an index (mask
    tensor, plan) likewise; between the two bit for bit unless lists are split
    or heads share a tile.  There both stay within the rounding of the weights
    (and at D = 128 of the scaled Q) to bf16, 2^-9 each, of the same result:
    2^-8 of the output's norm."""
    q, k, v = (t.cuda() for t in small_qkv(29, B, Hq, Hkv, S_q, S_k, D))
    plain, indexed = forms(q, k, v, causal)
    for group in (plain, indexed):
        first = next(iter(group.values()))
        for name, out in group.items():
            assert torch.equal(first, out), name
    a, b = plain["fwd"], indexed["mask"]
    if same:
        assert torch.equal(a, b)
    assert ((a - b).double().norm() / b.double().norm()).item() <= 2.0 ** -8
    for h in (slice(0, 1), slice(B - 1, B)):
        want = oracle.attention(q[h].cpu(), k[h].cpu(), v[h].cpu(), None, D ** -0.5, causal, 64)
        check(a[h], want, "no mask tensor")
        check(b[h], want, "mask tensor")


@pytest.mark.parametrize("B,Hq,Hkv,S_q,S_k", [
    # partial results of 32.5 MiB and more (slots of D = 128 times 64 rows), above
    # the fixed array's 32: shared tiles (the last unit a batch of its own), pairs
    (8, 32, 8, 16, 8192),
    (8, 16, 8, 64, 4096),
], ids=str)
def test_partial_results_in_batches(B, Hq, Hkv, S_q, S_k):
    """steel_attn_fwd_noalloc takes the units in batches where steel_attn_fwd
    takes them at once: bit for bit the same, every row written, and against the
    oracle where the second batch begins and ends."""
    D = 128
    g = torch.Generator(device="cuda").manual_seed(31)
    q, k, v = (torch.randn((B, h, n, D), generator=g, device="cuda").to(torch.bfloat16)
               for h, n in ((Hq, S_q), (Hkv, S_k), (Hkv, S_k)))
    s = steel()
    want = s.attn_fwd(q, k, v)
    out = torch.full((B, Hq, S_q, D), float("nan"), dtype=torch.float32, device="cuda")
    st = s._lib.load().steel_attn_fwd_noalloc(
        q.data_ptr(), k.data_ptr(), v.data_ptr(), None, out.data_ptr(), B, Hq, Hkv, S_q, S_k, D, 64,
        D ** -0.5, 1, torch.cuda.current_stream().cuda_stream)
    assert st == 0
    assert torch.isfinite(out).all()
    assert torch.equal(out, want)
    for g0 in (0, Hkv - 2, Hkv - 1):  # key/value groups of the last sequence
        hq = slice(g0 * (Hq // Hkv), (g0 + 1) * (Hq // Hkv))
        ref = oracle.attention(q[-1:, hq].cpu(), k[-1:, g0:g0 + 1].cpu(), v[-1:, g0:g0 + 1].cpu(), None,
                               D ** -0.5, True, 64)
        check(out[-1:, hq], ref, f"group {g0}")
