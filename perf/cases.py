"""Workloads whose time is tracked, each through the library's public entry points.

A case names the kind of call, its sizes and its options; ``listed`` holds the
tracked ones and ``draw`` gives further ones of the same ranges.  The shapes
are those of the paper's models and of the library's own workloads: BERT
attention (12 heads, D = 64), Llama-style grouped heads (32 query heads over
8 key/value heads, D = 64 and 128) and the 24-head long-sequence sparse
attention, from one head at S = 512 to S = 32768.

Kinds:
  dense        attn_fwd without a block mask
  bernoulli    attn_fwd with a random block mask per query head
  window_mask  attn_fwd with the window + sink block mask as a tensor
  window       attn_fwd_window (the same pattern from block coordinates)
  topk         attn_fwd with a top-k mean-pooled block mask
  topk_mask    topk_block_mask (the producer of that mask)
  plan         Plan.run on a plan of the window + sink pattern
  chunk        attn_fwd_lse over two key chunks and attn_merge of the parts
  fp8          attn_fwd_lse with E4M3 operands and a bf16 output

Inputs are N(0,1) in bf16 drawn on the GPU from the seed; the top-k kinds add
a shared rank-4 component to Q and K, as the library's long sparse workload
does, so that block scores differ in earnest.
"""
import math

import torch

import paper_2607_09385_amd as steel

BLK = 64


def _case(name, kind, B, Hq, Hkv, Sq, Sk, D, causal=True, p=0.0, win=0, sink=0, num=0, den=0,
          fp8=""):
    c = {"kind": kind, "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Sk": Sk, "D": D,
         "causal": bool(causal), "p": p, "win": win, "sink": sink, "num": num, "den": den,
         "fp8": fp8}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one head, the shortest sequence: what a call costs beyond its work
        _case("mha1_s512_d64", "dense", 1, 1, 1, 512, 512, 64),
        # BERT encoder layer: a batch of ragged sequences, no causal structure
        _case("bert_b8_mha12_s500_d64", "dense", 8, 12, 12, 500, 500, 64, causal=False),
        # dense causal prefill of a grouped-query layer
        _case("gqa32x8_s4096_d128", "dense", 1, 32, 8, 4096, 4096, 128),
        # block-sparse prefill, every query head with its own mask
        _case("gqa32x8_s8192_d128_bernoulli25", "bernoulli", 1, 32, 8, 8192, 8192, 128, p=0.25),
        # windowed prefill of a long sequence, mask handed over as a tensor
        _case("gqa32x8_s16384_d128_window", "window_mask", 1, 32, 8, 16384, 16384, 128, win=16,
              sink=1),
        # windowed prefill from coordinates, two sequences of an odd length
        _case("gqa32x8_b2_s2999_d128_window", "window", 2, 32, 8, 2999, 2999, 128, win=8, sink=1),
        # the largest: 24 heads, 32768 tokens, top 10% of the key blocks
        _case("mha24_s32768_d64_top10", "topk", 1, 24, 24, 32768, 32768, 64, num=1, den=10),
        # and the selection of those blocks
        _case("mha24_s32768_d64_top10_mask", "topk_mask", 1, 24, 24, 32768, 32768, 64, num=1,
              den=10),
        # one layer of many that share a plan, grouped heads of 64
        _case("gqa32x8_s8192_d64_plan", "plan", 1, 32, 8, 8192, 8192, 64, win=32, sink=1),
        # chunked prefill: new queries against a key cache held in two pieces
        _case("gqa32x8_q1000_k12000_d128_chunk", "chunk", 1, 32, 8, 1000, 12000, 128),
        # one decoding step of a batch against its key cache
        _case("gqa32x8_b4_q1_k8000_d128", "dense", 4, 32, 8, 1, 8000, 128),
        # fp8 operands, bf16 output
        _case("gqa32x8_s4096_d128_fp8", "fp8", 1, 32, 8, 4096, 4096, 128, fp8="all"),
    ]


_HEADS = {64: [(1, 1), (8, 8), (12, 12), (24, 24), (32, 8), (32, 32)],
          128: [(8, 2), (16, 4), (32, 8), (32, 32), (24, 6), (16, 8)]}


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _length(rng, lo, hi):
    s = _log(rng, lo, hi)
    return max(lo, s // BLK * BLK) if rng.random() < 0.5 else s  # whole blocks, or ragged


def _draw(rng):
    kind = rng.choice(["dense", "dense", "bernoulli", "window_mask", "window", "topk", "topk_mask",
                       "plan", "chunk", "decode", "fp8"])
    D = rng.choice([64, 128])
    Hq, Hkv = rng.choice(_HEADS[D])
    B = rng.choice([1, 1, 1, 2, 4, 8])
    if kind == "dense":
        s = _length(rng, 128, 8192)
        return _case("", kind, B, Hq, Hkv, s, s, D, causal=rng.random() < 0.7)
    if kind == "decode":
        return _case("", "dense", rng.choice([1, 2, 4, 8, 16]), Hq, Hkv, rng.choice([1, 1, 4, 17]),
                     _length(rng, 1024, 32768), D)
    if kind == "chunk":
        sq = _length(rng, 256, 4096)
        return _case("", kind, 1, Hq, Hkv, sq, sq + _length(rng, 1024, 24576), D)
    if kind == "bernoulli":
        s = _length(rng, 1024, 16384)
        return _case("", kind, B, Hq, Hkv, s, s, D, p=rng.choice([0.1, 0.25, 0.5]))
    if kind in ("window_mask", "window", "plan"):
        s = _length(rng, 1024, 32768)
        return _case("", kind, B, Hq, Hkv, s, s, D, win=rng.choice([4, 8, 16, 32]),
                     sink=rng.choice([0, 1, 2]))
    if kind in ("topk", "topk_mask"):
        s = _length(rng, 2048, 32768)
        return _case("", kind, 1, Hq, Hkv, s, s, D, num=1, den=rng.choice([4, 8, 10]))
    s = _length(rng, 512, 8192)
    return _case("", "fp8", B, Hq, Hkv, s, s, D, fp8=rng.choice(["all", "pv"]))


def draw(rng):
    most = [work(c) for c in listed()]
    flops, nbytes = max(w["flops"] for w in most), max(w["bytes"] for w in most)
    while True:
        c = _draw(rng)
        w = work(c)
        if w["flops"] <= flops and w["bytes"] <= nbytes:
            return c


# ---- what the cases' inputs are ----

def _blocks(s):
    return -(-s // BLK)


def _qkv(case, seed):
    dev = torch.device("cuda")
    g = torch.Generator(device=dev).manual_seed(int(seed))
    B, Hq, Hkv, Sq, Sk, D = (case[n] for n in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
    q = torch.randn((B, Hq, Sq, D), generator=g, device=dev)
    k = torch.randn((B, Hkv, Sk, D), generator=g, device=dev)
    v = torch.randn((B, Hkv, Sk, D), generator=g, device=dev)
    if case["kind"] in ("topk", "topk_mask"):  # shared rank-4 component of each key/value group
        u = torch.randn((B, Hkv, Sk, 4), generator=g, device=dev)
        w = torch.randn((B, Hkv, 4, D), generator=g, device=dev)
        low = u @ w
        k += low
        q += low.repeat_interleave(Hq // Hkv, dim=1)
    return tuple(t.to(torch.bfloat16).contiguous() for t in (q, k, v)), g


def _topk_mask(case, q, k):
    """Per query block the best ceil(num/den * candidates) key blocks by the
    float64 product of block means (equal scores: the smaller block), and the
    diagonal."""
    B, Hq, Hkv, S, D = case["B"], case["Hq"], case["Hkv"], case["Sq"], case["D"]
    n = _blocks(S)
    rows = torch.full((n,), float(BLK), dtype=torch.float64, device=q.device)
    rows[-1] = S - (n - 1) * BLK

    def means(x):
        pad = torch.zeros((x.shape[0], n * BLK, D), dtype=torch.float64, device=x.device)
        pad[:, :S] = x
        return pad.view(x.shape[0], n, BLK, D).sum(2) / rows[:, None]

    qb = torch.arange(n, device=q.device)
    ncand = qb + 1 if case["causal"] else torch.full_like(qb, n)
    keep = (case["num"] * ncand + case["den"] - 1) // case["den"]
    dead = qb[None, :] >= ncand[:, None]
    out = torch.empty((B, Hq, n, n), dtype=torch.uint8, device=q.device)
    for b in range(B):
        qm, km = means(q[b]), means(k[b])
        for h in range(Hq):
            sc = (qm[h] @ km[h // (Hq // Hkv)].T).masked_fill(dead, -math.inf)
            at = sc.sort(dim=1, descending=True, stable=True).indices
            rank = torch.empty_like(at).scatter_(1, at, qb[None, :].expand(n, n))
            live = (rank < keep[:, None]) & ~dead
            live[qb, qb] = True
            out[b, h] = live
    return out


def _mask(case, q, k, g):
    """The block mask as a tensor, or None where every block is in it."""
    B, Hq, nq, nk = case["B"], case["Hq"], _blocks(case["Sq"]), _blocks(case["Sk"])
    if case["kind"] == "bernoulli":
        m = torch.rand((B, Hq, nq, nk), generator=g, device=q.device) < case["p"]
        d = torch.arange(min(nq, nk), device=q.device)
        m[:, :, d, d] = True
        return m.to(torch.uint8)
    if case["win"]:
        i, j = torch.arange(nq, device=q.device)[:, None], torch.arange(nk, device=q.device)
        m = ((j <= i) & (j > i - case["win"])) | (j < case["sink"])
        return m.to(torch.uint8).expand(B, Hq, nq, nk).contiguous()
    if case["kind"] == "topk":
        return _topk_mask(case, q, k)
    return None


def _split(case):
    """First key of the second chunk: the cache before this chunk's own keys."""
    return case["Sk"] - case["Sq"]


def prepare(case, seed):
    (q, k, v), g = _qkv(case, seed)
    kind = case["kind"]
    st = {"case": case, "q": q, "k": k, "v": v, "scale": case["D"] ** -0.5}
    if kind in ("bernoulli", "window_mask", "topk"):
        st["mask"] = _mask(case, q, k, g)
    elif kind == "plan":
        st["plan"] = steel.Plan(None, case["B"], case["Hq"], case["Hkv"], case["Sq"], case["Sk"],
                                causal=case["causal"], window=(case["win"], case["sink"]))
    elif kind == "chunk":
        at = _split(case)
        st["parts"] = [(0, k[:, :, :at].contiguous(), v[:, :, :at].contiguous()),
                       (at, k[:, :, at:].contiguous(), v[:, :, at:].contiguous())]
        del st["k"], st["v"]
    return st


def run(st):
    case, q = st["case"], st["q"]
    kind, causal, scale = case["kind"], case["causal"], st["scale"]
    if kind == "window":
        return steel.attn_fwd_window(q, st["k"], st["v"], case["win"], case["sink"], scale=scale,
                                     causal=causal)
    if kind == "topk_mask":
        return steel.topk_block_mask(q, st["k"], case["num"], case["den"], causal=causal)
    if kind == "plan":
        return st["plan"].run(q, st["k"], st["v"], scale=scale)
    if kind == "fp8":
        out, lse = steel.attn_fwd_lse(q, st["k"], st["v"], scale=scale, causal=causal,
                                      out_dtype=torch.bfloat16, fp8=case["fp8"])
        return {"out": out, "lse": lse}
    if kind == "chunk":
        parts = st["parts"]
        o = torch.empty((len(parts),) + tuple(q.shape), dtype=torch.float32, device=q.device)
        l = torch.empty((len(parts),) + tuple(q.shape[:3]), dtype=torch.float32, device=q.device)
        for i, (at, k, v) in enumerate(parts):
            steel.attn_fwd_lse(q, k, v, scale=scale, causal=causal,
                               causal_offset=case["Sk"] - case["Sq"] - at, out=o[i], lse=l[i])
        out, lse = steel.attn_merge(o, l)
        return {"out": out, "lse": lse}
    return steel.attn_fwd(q, st["k"], st["v"], st.get("mask"), scale=scale, causal=causal)


# ---- what a pass cannot do without ----

def _visible(case):
    """Visible (query, key) pairs of one query head."""
    Sq, Sk, causal = case["Sq"], case["Sk"], case["causal"]
    nq, nk = _blocks(Sq), _blocks(Sk)
    delta = Sk - Sq
    if case["kind"] in ("dense", "chunk", "fp8"):
        if not causal:
            return float(Sq) * Sk
        return sum(min(max(i + delta + 1, 0), Sk) for i in range(Sq))
    total = 0.0
    for qb in range(nq):
        rows = min(BLK, Sq - qb * BLK)
        full = min(qb, nk) * BLK  # keys before the diagonal block (Sq == Sk)
        diag = rows * (rows + 1) / 2.0
        if case["kind"] == "bernoulli":
            total += case["p"] * full * rows + diag
        elif case["win"]:
            blocks = min(qb, max(case["win"] - 1, 0))
            blocks += min(case["sink"], qb - blocks)
            total += blocks * BLK * rows + diag
        else:  # top-k: the kept blocks, the diagonal among them or added
            keep = -(-case["num"] * (qb + 1) // case["den"])
            total += (min(keep, qb)) * BLK * rows + diag
    return total


def work(case):
    B, Hq, Hkv, Sq, Sk, D = (case[n] for n in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
    nq, nk = _blocks(Sq), _blocks(Sk)
    q, kv, rows = 2 * B * Hq * Sq * D, 2 * 2 * B * Hkv * Sk * D, B * Hq * Sq
    mask = B * Hq * nq * nk
    if case["kind"] == "topk_mask":
        pairs = nq * (nq + 1) / 2 if case["causal"] else nq * nk
        return {"bytes": q + kv // 2 + mask, "flops": 2.0 * B * Hq * pairs * D + rows * D}
    out = rows * D * (2 if case["kind"] == "fp8" else 4)
    nbytes = q + kv + out
    if case["kind"] in ("bernoulli", "window_mask", "topk"):
        nbytes += mask
    if case["kind"] in ("fp8", "chunk"):
        nbytes += rows * 4
    return {"bytes": nbytes, "flops": 4.0 * D * B * Hq * _visible(case)}


# ---- how close another correct implementation comes ----

def tolerance(case):
    if case["kind"] == "topk_mask":
        return "exact"  # the selection's arithmetic is fixed: a mask of bytes
    if case["kind"] == "fp8":
        # E4M3 weights (3 mantissa bits) round elsewhere under another running maximum
        return {"rel": 2e-2}
    return {"rel": 1e-2}  # bf16 operands and weights, 32-bit sums


def exact(case, seed):
    (q, k, v), g = _qkv(case, seed)
    if case["kind"] == "topk_mask":
        return _topk_mask(case, q, k)
    B, Hq, Hkv, Sq, Sk, D = (case[n] for n in ("B", "Hq", "Hkv", "Sq", "Sk", "D"))
    mask = _mask(case, q, k, g)
    out = torch.zeros((B, Hq, Sq, D), dtype=torch.float64, device=q.device)
    lse = torch.full((B, Hq, Sq), -math.inf, dtype=torch.float64, device=q.device)
    step = max(BLK, (1 << 27) // Sk // BLK * BLK)  # query rows at a time: 1 GiB of scores
    keys = torch.arange(Sk, device=q.device)
    for b in range(B):
        for h in range(Hq):
            kd, vd = k[b, h // (Hq // Hkv)].double(), v[b, h // (Hq // Hkv)].double()
            for r0 in range(0, Sq, step):
                r1 = min(r0 + step, Sq)
                s = (q[b, h, r0:r1].double() * case["D"] ** -0.5) @ kd.T
                if case["causal"]:
                    s.masked_fill_(keys[None, :] > torch.arange(r0, r1, device=q.device)[:, None]
                                   + (Sk - Sq), -math.inf)
                if mask is not None:
                    live = mask[b, h, r0 // BLK:_blocks(r1)].bool().repeat_interleave(BLK, 0)
                    live = live[: r1 - r0].repeat_interleave(BLK, 1)[:, :Sk]
                    s.masked_fill_(~live, -math.inf)
                top = s.amax(1, keepdim=True)
                top = torch.where(torch.isfinite(top), top, torch.zeros_like(top))
                s = torch.exp_(s - top)
                tot = s.sum(1, keepdim=True)
                out[b, h, r0:r1] = (s @ vd) / torch.where(tot > 0, tot, torch.ones_like(tot))
                lse[b, h, r0:r1] = (top + torch.log(tot))[:, 0]
    if case["kind"] in ("fp8", "chunk"):
        return {"out": out, "lse": lse}
    return out
