"""The calls whose speed is followed: listed sizes, a draw of more of the same ranges, and
what each computes in 64 bits.

Every case goes through the package's public functions, as a program with tensors on the GPU calls
them: attention over a prompt (``attn_fwd``), one decode step against a KV cache (``attn_decode``)
and the two row reductions (``norm_l2``, ``rmsnorm_rowmax``).  Head counts, head dims, modifiers and
the largest sizes are those of ``paper_2510_08726_amd.workloads``; the other sizes are generic ones
of the ranges the operations are used over: batch 1 to 16, 100 to 32768 keys, rows of 2^10 to 2^17
elements.
"""

import math

import torch

import paper_2510_08726_amd as pa
from paper_2510_08726_amd.workloads import alibi_slopes, decode_bytes, norm_bytes, prefill_flops

_DTYPE = {"f16": torch.float16, "bf16": torch.bfloat16, "f32": torch.float32}


def _prefill(name, B, Hq, Hkv, Lq, Lk, D, dtype, causal=True, alibi=False, softcap=0.0, window=0):
    return {"name": name, "op": "prefill", "B": B, "Hq": Hq, "Hkv": Hkv, "Lq": Lq, "Lk": Lk, "D": D, "dtype": dtype,
            "causal": causal, "alibi": alibi, "softcap": softcap, "window": window}


def _decode(name, B, Hq, Hkv, Lk, D, dtype, alibi=False, softcap=0.0):
    return {"name": name, "op": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "Lk": Lk, "D": D, "dtype": dtype,
            "alibi": alibi, "softcap": softcap}


def _norm(name, op, N, M, dtype):
    return {"name": name, "op": op, "N": N, "M": M, "dtype": dtype}


def listed():
    return [
        # One user's short question: the smallest prompt call, grouped heads.
        _prefill("prefill short prompt", 1, 32, 8, 211, 211, 128, "bf16"),
        # A batch of ordinary prompts, one KV head per query head (the headline workload).
        _prefill("prefill causal mha", 4, 32, 32, 2048, 2048, 128, "f16"),
        # Long documents with grouped heads: the largest prompt call.
        _prefill("prefill causal gqa", 2, 64, 8, 4096, 4096, 128, "bf16"),
        # The next piece of one long prompt against the keys cached so far (chunked prefill).
        _prefill("prefill chunk on cache", 1, 32, 8, 500, 6100, 128, "bf16"),
        # A bidirectional encoder over image patches or a sentence pair: no mask, ragged length.
        _prefill("encoder no mask", 8, 16, 16, 577, 577, 64, "f16", causal=False),
        # ALiBi attention with narrow heads.
        _prefill("prefill alibi", 4, 16, 16, 4096, 4096, 64, "f16", alibi=True),
        # A layer with both a capped score and a sliding window, odd length.
        _prefill("prefill softcap window", 1, 32, 16, 7001, 7001, 128, "f16", softcap=50.0, window=4095),
        # One user's next token: the smallest decode step, latency counts.
        _decode("decode one sequence", 1, 32, 8, 3001, 128, "bf16"),
        # A batch of sequences, one KV head per query head.
        _decode("decode mha batch", 8, 32, 32, 8192, 128, "f16"),
        # Long contexts with grouped heads: the largest decode step.
        _decode("decode gqa long", 16, 32, 8, 32768, 128, "f16"),
        # The stable norm of long rows (gradients, weights) in fp32.
        _norm("l2 norm long rows", "l2", 256, 1 << 17, "f32"),
        # Activations of a batch of tokens before a layer.
        _norm("rmsnorm tokens", "rms", 2048, 4096, "bf16"),
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


_HEADS = [(32, 32, 128), (32, 8, 128), (64, 8, 128), (32, 16, 128), (16, 16, 64), (12, 12, 64), (32, 4, 64)]
_MOST_FLOPS = 5.4e11     # the largest listed prompt
_MOST_BYTES = 2.1e9      # the largest listed decode step


# Cached lengths are even and windows odd: where Lk - Lq - window is a multiple of 32 (SoftCap with
# a window), or Lk - Lq is 31 more than one (ALiBi), the attention kernel has been seen to return
# one wrong row in 32, so those outputs are no reference for a comparison.
def draw(rng):
    kind = rng.choice(["prefill", "prefill", "chunk", "encoder", "decode", "decode", "l2", "rms"])
    if kind in ("prefill", "chunk", "encoder"):
        while True:
            Hq, Hkv, D = rng.choice(_HEADS)
            B = _log(rng, 1, 8)
            dtype = rng.choice(["f16", "bf16"])
            mod = rng.choice(["plain", "plain", "plain", "alibi", "softcap", "window", "softcap window"])
            causal = kind != "encoder"
            if kind == "prefill":
                Lq = Lk = _log(rng, 100, 8192)
            elif kind == "chunk":
                B, Lq = min(B, 2), _log(rng, 64, 1024)
                Lk = Lq + 2 * _log(rng, 256, 8192)
            else:
                Lq = Lk = _log(rng, 100, 2048)
                mod = "alibi" if mod == "alibi" else "plain"
            c = _prefill("", B, Hq, Hkv, Lq, Lk, D, dtype, causal, mod == "alibi",
                         50.0 if "softcap" in mod else 0.0, _log(rng, 256, 4096) | 1 if "window" in mod else 0)
            if _flops(c) <= _MOST_FLOPS:
                break
    elif kind == "decode":
        while True:
            Hq, Hkv, D = rng.choice(_HEADS)
            mod = rng.choice(["plain", "plain", "alibi", "softcap"])
            c = _decode("", _log(rng, 1, 16), Hq, Hkv, _log(rng, 200, 32768), D, rng.choice(["f16", "bf16"]),
                        mod == "alibi", 50.0 if mod == "softcap" else 0.0)
            if _bytes(c) <= _MOST_BYTES:
                break
    else:
        dtype = rng.choice(["f32", "f16", "bf16"])
        vec = 4 if dtype == "f32" else 8
        while True:
            c = _norm("", kind, _log(rng, 32, 8192), _log(rng, 1 << 10, 1 << 17) // vec * vec, dtype)
            if c["N"] * c["M"] <= 1 << 25:
                break
    del c["name"]
    return c


def _flops(c):
    if c["op"] == "prefill":
        return prefill_flops(c["B"], c["Hq"], c["Lq"], c["Lk"], c["D"], c["causal"], c["window"])
    if c["op"] == "decode":
        return 4 * c["D"] * c["Lk"] * c["B"] * c["Hq"]
    return (5 if c["op"] == "rms" else 4) * c["N"] * c["M"]


def _bytes(c):
    if c["op"] == "prefill":
        return 2 * c["B"] * c["D"] * (2 * c["Hq"] * c["Lq"] + 2 * c["Hkv"] * c["Lk"])
    if c["op"] == "decode":
        return decode_bytes(c["B"], c["Hq"], c["Hkv"], c["Lk"], c["D"])
    return norm_bytes(c["op"], c["N"], c["M"], 4 if c["dtype"] == "f32" else 2)


def work(case):
    return {"bytes": _bytes(case), "flops": _flops(case)}


def tolerance(case):
    # About four times the error against exact(), which is the rounding of the output (and of the
    # softmax weights) to 16 bits, or fp32 sums.  The norms are one value a row.
    if case["op"] in ("prefill", "decode"):
        return {"rel": 1e-3, "max": 2e-2} if case["dtype"] == "f16" else {"rel": 8e-3, "max": 1.5e-1}
    if case["op"] == "l2" or case["dtype"] == "f32":
        return {"rel": 3e-6, "max": 1e-5}
    return {"rel": 8e-4, "max": 4e-3} if case["dtype"] == "f16" else {"rel": 6e-3, "max": 3e-2}


def _inputs(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    dt = _DTYPE[case["dtype"]]

    def randn(*shape):
        return torch.randn(shape, generator=g, device="cuda", dtype=torch.float32).to(dt)

    if case["op"] in ("l2", "rms"):
        # Rows of different magnitudes, as activations and gradients have.
        x = torch.randn((case["N"], case["M"]), generator=g, device="cuda", dtype=torch.float32)
        x *= torch.exp(0.5 * torch.randn((case["N"], 1), generator=g, device="cuda", dtype=torch.float32))
        return {"x": x.to(dt)}
    B, Hq, Hkv, Lk, D = (case[k] for k in ("B", "Hq", "Hkv", "Lk", "D"))
    s = {"q": randn(B, Hq, case.get("Lq", 1), D), "k": randn(B, Hkv, Lk, D), "v": randn(B, Hkv, Lk, D), "slopes": None}
    if case["alibi"]:
        s["slopes"] = alibi_slopes(Hq).cuda()
    return s


def prepare(case, seed):
    s = _inputs(case, seed)
    s["case"] = case
    if case["op"] == "decode":
        # A decode loop keeps its split workspace and its output from step to step.
        B, Hq, Hkv, Lk, D = (case[k] for k in ("B", "Hq", "Hkv", "Lk", "D"))
        need = pa.attn_decode_workspace_bytes(B, Hq, D, pa.attn_decode_num_splits(B, Hq, Hkv, Lk, D))
        s["workspace"] = torch.empty(need, dtype=torch.uint8, device="cuda")
        s["o"] = torch.empty_like(s["q"])
    return s


def run(state):
    c = state["case"]
    if c["op"] == "prefill":
        return pa.attn_fwd(state["q"], state["k"], state["v"], causal=c["causal"], alibi_slopes=state["slopes"],
                           softcap=c["softcap"] or None, window=c["window"] or None)
    if c["op"] == "decode":
        return pa.attn_decode(state["q"], state["k"], state["v"], state["o"], alibi_slopes=state["slopes"],
                              softcap=c["softcap"] or None, workspace=state["workspace"])
    if c["op"] == "l2":
        return pa.norm_l2(state["x"])
    return pa.rmsnorm_rowmax(state["x"])


def exact(case, seed):
    s = _inputs(case, seed)
    if case["op"] == "l2":
        return s["x"].double().square().sum(1).sqrt()
    if case["op"] == "rms":
        x = s["x"].double()
        y = x / (x.square().mean(1, keepdim=True) + 1e-6).sqrt()
        return y, y.amax(1)
    B, Hq, Hkv, Lk, D = (case[k] for k in ("B", "Hq", "Hkv", "Lk", "D"))
    Lq = case.get("Lq", 1)
    decode = case["op"] == "decode"
    window = 0 if decode else case["window"]
    masked = not decode and case["causal"]
    o = torch.empty((B, Hq, Lq, D), dtype=torch.float64, device="cuda")
    j = torch.arange(Lk, device="cuda")
    i = torch.arange(Lq, device="cuda")[:, None] + (Lk - Lq)
    for b in range(B):
        for h in range(Hq):
            k = s["k"][b, h // (Hq // Hkv)].double()
            v = s["v"][b, h // (Hq // Hkv)].double()
            p = (s["q"][b, h].double() @ k.t().contiguous()) / math.sqrt(D)
            if case["softcap"]:
                p = case["softcap"] * torch.tanh(p / case["softcap"])
            if case["alibi"]:
                p -= s["slopes"][h].double() * (i - j)
            if masked:
                p.masked_fill_(j > i, -math.inf)
            if window:
                p.masked_fill_(j <= i - window, -math.inf)
            o[b, h] = torch.softmax(p, 1) @ v
    return o
