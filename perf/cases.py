"""The calls whose speed is measured: attention layers as a program runs them.

Each case is one attention layer through the package's public entry points:

* ``fwd``: ``attn_fwd`` (inference; the output is allocated by the call),
* ``lse``: ``attn_fwd_lse`` (a forward whose statistics the program keeps),
* ``persistent``: ``attn_fwd_persistent`` with a queue that the program keeps,
* ``train``: ``attn_fwd_lse`` and ``attn_bwd``, the layer's part of a step.

Inputs are i.i.d. N(0, 1) rounded to bf16, as everywhere in this repository,
scale 1/sqrt(d).
"""

from __future__ import annotations

import math

import torch

import paper_2511_02132_amd as pa

DEV = "cuda:0"


def _case(name, call, B, Hq, Hkv, Sq, Skv, d, causal, mapping):
    return {"name": name, "call": call, "B": B, "Hq": Hq, "Hkv": Hkv, "Sq": Sq, "Skv": Skv,
            "d": d, "causal": causal, "mapping": mapping}


# Placements in use: the paper's swizzled head-first, with each head's heaviest
# row blocks first under a causal mask (the package's method_variant).
SHF = pa.SWIZZLED_HEAD_FIRST
SHF_HF = pa.SWIZZLED_HEAD_FIRST | pa.HEAVY_FIRST
SHF_HF_BM = pa.SWIZZLED_HEAD_FIRST | pa.HEAVY_FIRST | pa.XCD_BLOCK_MAJOR
NBF_HF = pa.NAIVE_BLOCK_FIRST | pa.HEAVY_FIRST


def listed():
    return [
        # a small encoder layer, the smallest workload: launch latency counts
        _case("short_mha_b1_h4_s256_d64", "fwd", 1, 4, 4, 256, 256, 64, False, SHF),
        # one decoding step of a 70B-class GQA layer over an 8K cache, batch 4
        _case("decode_gqa_b4_h64_kv8_s8192_d128", "fwd", 4, 64, 8, 1, 8192, 128, False, SHF),
        # an 8B-class layer's prefill of one ordinary prompt (ragged length)
        _case("prefill_mha_b1_h32_s1000_d128", "fwd", 1, 32, 32, 1000, 1000, 128, True, SHF_HF),
        # the same layer's prefill of a long prompt
        _case("prefill_mha_b1_h32_s8192_d128", "fwd", 1, 32, 32, 8192, 8192, 128, True, SHF_HF),
        # a 70B-class GQA layer's prefill in the dispatch-independent form
        _case("persistent_gqa_b1_h64_kv8_s8192_d128", "persistent", 1, 64, 8, 8192, 8192, 128,
              True, SHF_HF),
        # batched bidirectional attention
        _case("encode_mha_b8_h64_s4096_d128", "fwd", 8, 64, 64, 4096, 4096, 128, False, SHF),
        # a 128K-token context, the largest workload
        _case("prefill_mha_b1_h16_s131072_d128", "fwd", 1, 16, 16, 131072, 131072, 128, True,
              SHF_HF),
        # DeepSeek-V3-shaped heads, a 2K prompt
        _case("prefill_mha_b1_h128_s2048_d56", "fwd", 1, 128, 128, 2048, 2048, 56, True, SHF_HF),
        # batched d = 64 encoder layer of odd length whose statistics are kept
        _case("encode_lse_mha_b4_h16_s1500_d64", "lse", 4, 16, 16, 1500, 1500, 64, False, SHF),
        # training step of a small layer, ragged length
        _case("train_mha_b2_h16_s1111_d128", "train", 2, 16, 16, 1111, 1111, 128, True, SHF_HF),
        # training step of a GQA layer
        _case("train_gqa_b1_h32_kv8_s4096_d128", "train", 1, 32, 8, 4096, 4096, 128, True,
              SHF_HF),
        # training step of an 8B-class layer on long sequences
        _case("train_mha_b1_h32_s8192_d128", "train", 1, 32, 32, 8192, 8192, 128, True, SHF_HF),
    ]


_HEADS = [(4, 4), (8, 8), (16, 16), (32, 32), (64, 64), (12, 4), (16, 4), (32, 8), (64, 8), (8, 1)]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    """One more case: short, decoding, prefill, encoding or training calls."""
    while True:
        kind = rng.choice(["short", "decode", "prefill", "encode", "train"])
        Hq, Hkv = rng.choice(_HEADS)
        d = rng.choice([64, 128, 128, 56]) if kind != "train" else 128
        call, causal = "fwd", False
        if kind == "short":         # a few hundred rows
            B, Sq = rng.choice([1, 1, 2, 3]), _log_int(rng, 17, 700)
            Skv, causal = Sq, rng.random() < 0.5
        elif kind == "decode":      # one or a few new rows against a cache
            B, Sq, Skv = _log_int(rng, 1, 32), rng.choice([1, 1, 1, 2, 5, 8]), _log_int(rng, 300, 40000)
        elif kind == "prefill":
            B, Sq = rng.choice([1, 1, 2, 4]), _log_int(rng, 500, 20000)
            Skv, causal = Sq, True
        elif kind == "encode":      # self- or cross-attention without a mask
            B, Sq = rng.choice([1, 2, 4, 8]), _log_int(rng, 300, 6000)
            Skv = Sq if rng.random() < 0.6 else _log_int(rng, 64, 6000)
        else:
            call, B, Sq = "train", rng.choice([1, 2, 4]), _log_int(rng, 300, 8192)
            Skv, causal = Sq, rng.random() < 0.8
        if kind in ("prefill", "encode"):
            call = rng.choice(["fwd", "fwd", "lse", "persistent"] if d == 128 else ["fwd", "lse"])
        mapping = rng.choice([SHF_HF, SHF_HF, SHF_HF_BM, NBF_HF, SHF]) if causal else SHF
        case = _case("", call, B, Hq, Hkv, Sq, Skv, d, causal, mapping)
        del case["name"]
        cost = work(case)
        if cost["flops"] <= 8e12 and cost["bytes"] <= 4e9:
            return case


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))

    def rand(*shape):
        t = torch.empty(shape, dtype=torch.bfloat16, device=DEV)
        for row in t.view(-1, shape[-2], shape[-1]).split(64):   # drawn in fp32, in pieces
            row.copy_(torch.randn(row.shape, generator=g, device=DEV, dtype=torch.float32))
        return t

    c = case
    state = {"case": dict(c),
             "q": rand(c["B"], c["Hq"], c["Sq"], c["d"]),
             "k": rand(c["B"], c["Hkv"], c["Skv"], c["d"]),
             "v": rand(c["B"], c["Hkv"], c["Skv"], c["d"])}
    if c["call"] == "train":
        state["dout"] = rand(c["B"], c["Hq"], c["Sq"], c["d"])
    if c["call"] == "persistent":
        state["queue"] = pa.new_queue(DEV)
    return state


def run(state):
    c, q, k, v = state["case"], state["q"], state["k"], state["v"]
    opt = {"causal": c["causal"], "mapping": c["mapping"]}
    if c["call"] == "fwd":
        return pa.attn_fwd(q, k, v, **opt)
    if c["call"] == "lse":
        return pa.attn_fwd_lse(q, k, v, **opt)
    if c["call"] == "persistent":
        return pa.attn_fwd_persistent(q, k, v, queue=state["queue"], **opt)
    o, lse = pa.attn_fwd_lse(q, k, v, **opt)
    dq, dk, dv = pa.attn_bwd(q, k, v, o, state["dout"], lse, **opt)
    return o, lse, dq, dk, dv


def _pairs(Sq, Skv, causal):
    """(query row, key) pairs that the mask leaves."""
    if not causal:
        return Sq * Skv
    full = max(0, Sq - Skv)           # rows that see every key
    n = Sq - full
    return n * (n + 1) // 2 + full * Skv


def work(case):
    c = case
    qo = 2 * c["B"] * c["Hq"] * c["Sq"] * c["d"]
    kv = 2 * c["B"] * c["Hkv"] * c["Skv"] * c["d"]
    stat = 4 * c["B"] * c["Hq"] * c["Sq"]
    flops = 4 * c["B"] * c["Hq"] * _pairs(c["Sq"], c["Skv"], c["causal"]) * c["d"]
    nbytes = 2 * qo + 2 * kv
    if c["call"] == "lse":
        nbytes += stat
    if c["call"] == "train":          # dO in; lse, dQ, dK, dV out; two and five products
        nbytes += stat + 2 * qo + 2 * kv
        flops += 5 * flops // 2
    return {"bytes": nbytes, "flops": flops}


def tolerance(case):
    """Probabilities enter the matrix cores as bf16 and results leave as bf16:
    2^-9 relative for each rounding."""
    return {"rel": 1e-2}


def exact(case, seed):
    """The same outputs in float64 (torch on the same device), row blocks at a time."""
    c = case
    if work(c)["flops"] > 2e13:
        return None
    s = prepare(c, seed)
    B, Hq, Hkv, Sq, Skv, d = (c[x] for x in ("B", "Hq", "Hkv", "Sq", "Skv", "d"))
    scale, group = 1.0 / math.sqrt(d), Hq // Hkv
    train = c["call"] == "train"
    f64 = {"dtype": torch.float64, "device": DEV}
    o = torch.empty(B, Hq, Sq, d, **f64)
    lse = torch.empty(B, Hq, Sq, **f64)
    if train:
        dq, dk, dv = torch.zeros(B, Hq, Sq, d, **f64), torch.zeros(B, Hkv, Skv, d, **f64), \
            torch.zeros(B, Hkv, Skv, d, **f64)
    rows = max(1, min(Sq, 2 ** 25 // Skv))
    for b in range(B):
        for g in range(Hkv):
            k, v = s["k"][b, g].double(), s["v"][b, g].double()
            kt, vt = k.t().contiguous(), v.t().contiguous()
            for h in range(g * group, (g + 1) * group):
                for r0 in range(0, Sq, rows):
                    r1 = min(Sq, r0 + rows)
                    n = min(Skv, r1) if c["causal"] else Skv
                    q = s["q"][b, h, r0:r1].double()
                    x = (q @ kt[:, :n]) * scale
                    if c["causal"]:
                        i = torch.arange(r0, r1, device=DEV)[:, None]
                        x.masked_fill_(torch.arange(n, device=DEV)[None, :] > i, -math.inf)
                    lse[b, h, r0:r1] = torch.logsumexp(x, dim=1)
                    p = torch.exp(x - lse[b, h, r0:r1, None])
                    ob = p @ v[:n]
                    o[b, h, r0:r1] = ob
                    if train:
                        do = s["dout"][b, h, r0:r1].double()
                        dv[b, g, :n] += p.t().contiguous() @ do
                        ds = p * (do @ vt[:, :n] - (do * ob).sum(1, keepdim=True))
                        dq[b, h, r0:r1] = scale * (ds @ k[:n])
                        dk[b, g, :n] += scale * (ds.t().contiguous() @ q)
    if train:
        return o, lse, dq, dk, dv
    return (o, lse) if c["call"] == "lse" else o
