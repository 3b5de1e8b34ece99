"""Timing cases of the attention library: what its users call, over the sizes they call it with.

A case is a dict of plain values:
  kind     "train"  attention() forward and backward through autograd
           "gqa"    the same with fewer key/value heads than query heads
           "chunk"  forward only, few queries against a longer context (attn_fwd_rect)
           "stats"  the rounding-bias measurement of one layer: forward with its float32 output and
                    tie counts, delta from both outputs, dQ with either delta (what harness.run does
                    between its projections)
  B, H, Hkv, Nq, Nk, d, causal, variant (0 Alg. 1, 1 Alg. 3 per tile, 2 Alg. 3 on whole rows)
  layout   "bhnd" contiguous [B,H,N,d], or "fused": q, k, v are views into one [B,N,3,H,d] projection
  scale    multiplies the N(0,1) draws of Q and K (1: flat softmax, 2: sharp)
"""
import math

import torch

from paper_2510_04212_amd import binding
from paper_2510_04212_amd.autograd import attention

DEV = "cuda:0"


def _case(name, kind, B, H, Nq, d, causal, variant, Nk=None, Hkv=None, layout="bhnd", scale=1.0):
    c = {"kind": kind, "B": B, "H": H, "Hkv": Hkv or H, "Nq": Nq, "Nk": Nk or Nq, "d": d,
         "causal": causal, "variant": variant, "layout": layout, "scale": scale}
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # one short sequence, one head: latency and launches (unit tests, debugging, probing models)
        _case("tiny", "train", 1, 1, 128, 64, False, 0),
        # GPT-2-small attention (the paper's training setting), q, k, v straight from the fused projection
        _case("gpt2s", "train", 8, 12, 1024, 64, True, 1, layout="fused", scale=1.5),
        # mid-scale training shape, the headline throughput case
        _case("mid", "train", 4, 32, 4096, 128, True, 1),
        # long context, sharp attention
        _case("long", "train", 1, 16, 16384, 128, True, 1, scale=2.0),
        # a sequence length that no tile divides
        _case("ragged", "train", 4, 16, 1999, 128, True, 1),
        # bidirectional encoder: many short sequences, no mask, plain softmax
        _case("encoder", "train", 32, 12, 512, 64, False, 0),
        # grouped-query attention, four query heads to a key/value head
        _case("gqa", "gqa", 2, 32, 2048, 128, True, 1, Hkv=8),
        # a chunk of new queries against a cached context
        _case("chunk", "chunk", 2, 16, 64, 128, True, 1, Nk=8192),
        # the two head sizes of larger and odder models
        _case("d96", "train", 2, 16, 2048, 96, True, 1),
        _case("d256", "train", 2, 8, 2048, 256, True, 1),
        # Alg. 3 decided on whole rows
        _case("row", "train", 4, 12, 1024, 64, True, 2, scale=1.5),
        # one step of the bias measurement
        _case("stats", "stats", 4, 12, 1024, 64, True, 0, scale=1.5),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the same ranges.  At most a third of the largest listed case's arithmetic
    (the head sizes that are not 128 run at a lower rate)."""
    while True:
        kind = rng.choice(["train"] * 5 + ["gqa", "gqa", "chunk", "chunk", "stats"])
        d = rng.choice([64, 64, 128, 128, 128, 32, 96, 256])
        causal = rng.random() < 0.75
        variant = rng.choice([0, 1, 1, 1, 2]) if kind == "train" else rng.choice([0, 1])
        N = _log_int(rng, 64, 16384)
        if rng.random() < 0.6:
            N = max(128, N // 128 * 128)          # most programs pad to a round length; the others stay odd
        H = rng.choice([1, 4, 8, 12, 16, 32])
        B = _log_int(rng, 1, 64)
        Hkv, Nq, layout = H, N, "bhnd"
        if kind == "gqa":
            Hkv = H // rng.choice([g for g in (2, 4, 8) if H % g == 0] or [1])
        elif kind == "chunk":
            N = max(N, 512)
            Nq = min(N, _log_int(rng, 1, 512))
        elif kind == "train" and variant != 2 and rng.random() < 0.4:
            layout = "fused"
        c = _case(None, kind, B, H, Nq, d, causal, variant, Nk=N, Hkv=Hkv, layout=layout,
                  scale=rng.choice([1.0, 1.5, 2.0]))
        rows = B * H * max(Nq, N) * d
        if work(c)["flops"] <= 1.3e12 and rows <= 1 << 27:
            return c


def _randn(gen, shape, scale=1.0):
    return (scale * torch.randn(shape, generator=gen, device=DEV)).to(torch.bfloat16)


def prepare(case, seed):
    g = torch.Generator(device=DEV)
    g.manual_seed(int(seed))
    B, H, Hkv, Nq, Nk, d = (case[k] for k in ("B", "H", "Hkv", "Nq", "Nk", "d"))
    sc = case["scale"]
    if case["layout"] == "fused":
        qkv = torch.randn((B, Nq, 3, H, d), generator=g, device=DEV)
        qkv[:, :, :2] *= sc
        qkv = qkv.to(torch.bfloat16)
        q, k, v = (qkv[:, :, i].permute(0, 2, 1, 3) for i in range(3))
        # the gradient of the output projection's input arrives in that projection's layout
        do = _randn(g, (B, Nq, H, d)).permute(0, 2, 1, 3)
    else:
        q = _randn(g, (B, H, Nq, d), sc)
        k = _randn(g, (B, Hkv, Nk, d), sc)
        v = _randn(g, (B, Hkv, Nk, d))
        do = _randn(g, (B, H, Nq, d))
    if case["kind"] == "stats":
        # every key twice and values of one sign: the repeated row maxima the measurement is about
        k[:, :, 1::2] = k[:, :, 0:Nk - 1:2] if Nk % 2 else k[:, :, 0::2]
        v = -v.abs()
    s = {"q": q, "k": k, "v": v, "do": do, "alpha": 1.0 / math.sqrt(d), "case": dict(case)}
    if case["kind"] in ("train", "gqa"):
        for n in "qkv":
            s[n] = s[n].detach().requires_grad_(True)
    return s


def run(s):
    c, q, k, v = s["case"], s["q"], s["k"], s["v"]
    if c["kind"] in ("train", "gqa"):
        o = attention(q, k, v, causal=c["causal"], variant=c["variant"])
        dq, dk, dv = torch.autograd.grad(o, (q, k, v), s["do"])
        return {"o": o.detach(), "dq": dq, "dk": dk, "dv": dv}
    if c["kind"] == "chunk":
        o, lse = binding.attn_fwd_rect(q, k, v, c["causal"], s["alpha"], c["variant"])
        return {"o": o, "lse": lse}
    f = binding.attn_fwd_opt(q, k, v, c["causal"], s["alpha"], c["variant"], want_O_hp=True, want_counts=True)
    d_lp = binding.attn_delta(f["O"], s["do"])
    d_hp = binding.attn_delta_hp(f["O_hp"], s["do"])
    dq = [binding.attn_bwd_dq(q, k, v, s["do"], f["LSE"], d, c["causal"], s["alpha"]) for d in (d_lp, d_hp)]
    return {"f": f, "d_lp": d_lp, "d_hp": d_hp, "dq_lp": dq[0], "dq_hp": dq[1]}


def work(case):
    B, H, Hkv, Nq, Nk, d = (case[k] for k in ("B", "H", "Hkv", "Nq", "Nk", "d"))
    shift = Nk - Nq
    if not case["causal"]:
        seen = Nq * Nk
    else:                                     # query r sees keys 0 .. r + shift (shift >= 0 here)
        seen = Nq * (shift + 1) + Nq * (Nq - 1) // 2
    # a product over the visible (query, key) pairs costs 2 d flops per pair
    products = {"train": 7, "gqa": 7, "chunk": 2, "stats": 2 + 3 + 3}[case["kind"]]
    rows_q, rows_k = B * H * Nq, B * Hkv * Nk
    if case["kind"] == "chunk":
        nbytes = 2 * d * (2 * rows_q + 2 * rows_k) + 4 * rows_q
    elif case["kind"] == "stats":             # q, k, v, do in; O, dQ twice, O_hp, LSE, two counts, two deltas out
        nbytes = 2 * d * (5 * rows_q + 2 * rows_k) + 4 * d * rows_q + 20 * rows_q
    else:                                     # q, do, k, v in; o, dq, dk, dv out
        nbytes = 2 * d * (4 * rows_q + 4 * rows_k)
    return {"bytes": nbytes, "flops": 2 * d * products * B * H * seen}


def tolerance(case):
    """About four times what the results were seen to be off from the same path in 64 bits:
    rel 2.3e-3 .. 4.5e-3 for outputs and gradients (bf16 roundings of P, dS and the results), max up
    to 0.17 (first rows under the mask, where a gradient is a small difference of large terms)."""
    if case["kind"] == "stats":
        # dQ from the delta of the rounded output carries that output's rounding bias (seen: rel 7e-3);
        # a probability next to 1 may round either way, and a score next to the threshold of Alg. 3
        return {"rel": 2.5e-2, "max": 0.6, "differ": 2e-3}
    return {"rel": 1.2e-2, "max": 0.6}
