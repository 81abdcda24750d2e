"""Performance cases: the attention calls a program makes of this library.

Training (attn_fwd_bwd, and attn_fwd / attn_bwd where the two directions are
called apart), prompt processing (attn_fwd) and token generation
(attn_decode over a KV cache with grouped query heads), each from the
smallest call, where latency and launches count, to the largest. Sizes are
those of the workload tables in ``workloads`` and generic ones around them:
lengths that are no multiple of any tile, few and many heads, the head
dimensions 32, 64 and 128, both masks, bfloat16 and float32. The naive
(materialising) and the atomic-dQ paths are comparison realisations of the
same computation and are left to the benchmark.
"""
from __future__ import annotations

import math

import torch

import paper_2609_33916_amd as lib

DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
# time of one float32 product against one bfloat16 product on the matrix cores
F32_COST = 16


def _attn(name, do, B, H, n, d, dtype, causal, sigma_qk=1.0, sigma_do=1.0):
    return {"name": name, "do": do, "B": B, "H": H, "n": n, "d": d, "dtype": dtype, "causal": causal,
            "sigma_qk": sigma_qk, "sigma_do": sigma_do}


def _decode(name, B, Hq, Hkv, n, d, ragged):
    return {"name": name, "do": "decode", "B": B, "Hq": Hq, "Hkv": Hkv, "n": n, "d": d, "ragged": ragged}


def listed():
    return [
        # one user's next token: a short cache, four query heads per cache head
        _decode("decode_b1_hq32_n1000_d128", 1, 32, 8, 1000, 128, False),
        # a serving batch whose sequences have different lengths
        _decode("decode_b32_hq32_n4096_d128_ragged", 32, 32, 8, 4096, 128, True),
        # a large serving batch of long sequences
        _decode("decode_b16_hq64_n8192_d128", 16, 64, 8, 8192, 128, False),
        # prompt of one short request (inference only)
        _attn("fwd_b1h8_n333_d64_bf16_causal", "fwd", 1, 8, 333, 64, "bf16", True),
        # prompt of one long request (inference only)
        _attn("fwd_b1h32_n4096_d128_bf16_causal", "fwd", 1, 32, 4096, 128, "bf16", True),
        # the smallest training call: one head, one tile
        _attn("fwdbwd_b1h1_n128_d32_f32", "fwd_bwd", 1, 1, 128, 32, "f32", False),
        # float32 training of a small model
        _attn("fwdbwd_b4h8_n1024_d64_f32", "fwd_bwd", 4, 8, 1024, 64, "f32", False),
        # training on a small batch, length no multiple of a tile
        _attn("fwdbwd_b2h8_n1000_d128_bf16_causal", "fwd_bwd", 2, 8, 1000, 128, "bf16", True, 1.0, 0.1),
        # backward of an autograd function whose forward ran before (encoder, no mask)
        _attn("bwd_b4h12_n1537_d64_bf16", "bwd", 4, 12, 1537, 64, "bf16", False),
        # the table's training workloads: many heads at moderate length, causal ...
        _attn("fwdbwd_b8h16_n4096_d64_bf16_causal", "fwd_bwd", 8, 16, 4096, 64, "bf16", True, 1.0, 0.1),
        # ... and without a mask, with peaked rows ...
        _attn("fwdbwd_b16h32_n2048_d128_bf16_peaked", "fwd_bwd", 16, 32, 2048, 128, "bf16", False, 2.0, 1.0),
        # ... and the long-context one, the largest
        _attn("fwdbwd_b2h32_n16384_d128_bf16_causal", "fwd_bwd", 2, 32, 16384, 128, "bf16", True, 1.0, 0.1),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _cost(case):
    w = work(case)
    return w["flops"] * (F32_COST if case.get("dtype") == "f32" else 1)


def draw(rng):
    """One more call of the listed ones' ranges: any length, heads and batch."""
    if rng.random() < 0.3:
        while True:
            Hkv, G = rng.choice([1, 2, 4, 8]), rng.choice([1, 2, 4, 8])
            case = {"do": "decode", "B": _log_int(rng, 1, 32), "Hq": Hkv * G, "Hkv": Hkv,
                    "n": _log_int(rng, 64, 131072), "d": rng.choice([64, 128, 128]), "ragged": rng.random() < 0.5}
            if work(case)["bytes"] <= 5.4e8:
                return case
    largest = max(_cost(c) for c in listed())
    while True:
        dtype = rng.choice(["bf16", "bf16", "bf16", "f32"])
        case = {"do": rng.choice(["fwd", "fwd_bwd", "fwd_bwd", "bwd"]), "B": _log_int(rng, 1, 16),
                "H": _log_int(rng, 1, 32), "n": _log_int(rng, 64, 16384), "d": rng.choice([32, 64, 64, 128, 128, 128]),
                "dtype": dtype, "causal": rng.random() < 0.6, "sigma_qk": rng.choice([1.0, 2.0]),
                "sigma_do": rng.choice([0.1, 1.0])}
        if _cost(case) <= largest:
            return case


# ------------------------------------------------------------------ inputs --
def _inputs(case, seed):
    """Seeded inputs on the GPU; a decode cache has room for one more row than
    the longest sequence, and holds other values past each sequence's end."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(int(seed))

    def normal(shape, dtype, sigma=1.0):
        return (torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * sigma).to(dtype)

    if case["do"] == "decode":
        B, Hq, Hkv, n, d = (case[k] for k in ("B", "Hq", "Hkv", "n", "d"))
        bf16 = torch.bfloat16
        t = {"q": normal((B, Hq, d), bf16), "k_new": normal((B, Hkv, d), bf16), "v_new": normal((B, Hkv, d), bf16),
             "k_cache": normal((B, Hkv, n + 1, d), bf16), "v_cache": normal((B, Hkv, n + 1, d), bf16)}
        t["lens"] = _lens(case, gen)
        return t
    shape, dtype = (case["B"], case["H"], case["n"], case["d"]), DTYPES[case["dtype"]]
    return {"q": normal(shape, dtype, case["sigma_qk"]), "k": normal(shape, dtype, case["sigma_qk"]),
            "v": normal(shape, dtype), "do": normal(shape, dtype, case["sigma_do"])}


def _lens(case, gen):
    """Tokens cached per sequence: n, or between n / 2 and n with the first at n."""
    B, n = case["B"], case["n"]
    lens = torch.full((B,), n, dtype=torch.int32, device="cuda")
    if case["ragged"]:
        lens = torch.randint(n // 2, n + 1, (B,), generator=gen, device="cuda", dtype=torch.int32)
        lens[0] = n
    return lens


def prepare(case, seed):
    t = _inputs(case, seed)
    if case["do"] == "bwd":   # the forward's results, as autograd saves them
        t["o"], t["lse"] = lib.attn_fwd(t["q"], t["k"], t["v"], causal=case["causal"])
    t["case"] = case
    return t


def run(state):
    case = state["case"]
    if case["do"] == "decode":
        # the caches come back too: the step writes its new row into them
        o, lse = lib.attn_decode(state["q"], state["k_cache"], state["v_cache"], state["k_new"], state["v_new"],
                                 cache_lens=state["lens"], n=case["n"])
        return o, lse, state["k_cache"], state["v_cache"]
    q, k, v = state["q"], state["k"], state["v"]
    if case["do"] == "fwd":
        return lib.attn_fwd(q, k, v, causal=case["causal"])
    if case["do"] == "bwd":
        return lib.attn_bwd(q, k, v, state["o"], state["lse"], state["do"], causal=case["causal"])
    return lib.attn_fwd_bwd(q, k, v, state["do"], causal=case["causal"])


# -------------------------------------------------------------------- work --
def work(case):
    if case["do"] == "decode":
        B, Hq, Hkv, n, d = (case[k] for k in ("B", "Hq", "Hkv", "n", "d"))
        rows = B * n * (0.75 if case["ragged"] else 1.0)
        # cached rows read once, new rows read and written once, q read, O and L written
        return {"bytes": 4 * Hkv * d * rows + 8 * B * Hkv * d + 4 * B * Hq * d + 4 * B * Hq,
                "flops": 4 * Hq * d * rows}
    n, d, heads = case["n"], case["d"], case["B"] * case["H"]
    e = 2 if case["dtype"] == "bf16" else 4
    pairs = n * (n + 1) // 2 if case["causal"] else n * n
    # products per pair and tensors of n x d moved once: Q, K, V -> O; Q, K, V,
    # O, dO -> dQ, dK, dV (S recomputed); Q, K, V, dO -> O, dQ, dK, dV
    products, tensors = {"fwd": (2, 4), "bwd": (5, 8), "fwd_bwd": (7, 8)}[case["do"]]
    return {"bytes": heads * (tensors * n * d * e + 4 * n), "flops": 2 * products * d * pairs * heads}


# --------------------------------------------------------------- tolerance --
def tolerance(case):
    # About four times the measured error against 64 bits: in bfloat16 the
    # results (and P and dS as product operands) are rounded to 8 bits, 2.0e-3
    # to 2.8e-3 of a tensor's norm; in float32, 0.3e-6 to 1.2e-6
    return {"rel": 5e-6 if case.get("dtype") == "f32" else 1e-2}


# ------------------------------------------------------------------- exact --
def exact(case, seed):
    t = _inputs(case, seed)
    if case["do"] == "decode":
        return _exact_decode(case, t)
    n, d, causal, do = case["n"], case["d"], case["causal"], case["do"]
    heads, scale = case["B"] * case["H"], 1.0 / math.sqrt(case["d"])
    x = {k: a.reshape(heads, n, d) for k, a in t.items()}
    shape = (case["B"], case["H"], n, d)
    out = {k: torch.empty((heads, n, d), dtype=torch.float64, device="cuda") for k in ("o", "dq", "dk", "dv")}
    lse = torch.empty((heads, n), dtype=torch.float64, device="cuda")
    mask = torch.ones(n, n, dtype=torch.bool, device="cuda").triu_(1) if causal else None
    for i in range(heads):
        q, k, v, g = (x[key][i].double() for key in ("q", "k", "v", "do"))
        s = (q @ k.t()).mul_(scale)
        if causal:
            s.masked_fill_(mask, -math.inf)
        lse[i] = torch.logsumexp(s, 1)
        p = s.sub_(lse[i][:, None]).exp_()
        o = p @ v
        out["o"][i] = o
        if do != "fwd":
            out["dv"][i] = p.t() @ g
            ds = (g @ v.t()).sub_((o * g).sum(1)[:, None]).mul_(p).mul_(scale)
            out["dq"][i] = ds @ k
            out["dk"][i] = ds.t() @ q
    o, dq, dk, dv = (out[key].view(shape) for key in ("o", "dq", "dk", "dv"))
    lse = lse.view(shape[:3])
    return {"fwd": (o, lse), "bwd": (dq, dk, dv), "fwd_bwd": (o, lse, dq, dk, dv)}[do]


def _exact_decode(case, t):
    B, Hq, Hkv, d = (case[k] for k in ("B", "Hq", "Hkv", "d"))
    G, scale = Hq // Hkv, 1.0 / math.sqrt(d)
    o = torch.empty((B, Hq, d), dtype=torch.float64, device="cuda")
    lse = torch.empty((B, Hq), dtype=torch.float64, device="cuda")
    lens = t["lens"].tolist()
    for b in range(B):
        T = lens[b]
        t["k_cache"][b, :, T] = t["k_new"][b]
        t["v_cache"][b, :, T] = t["v_new"][b]
        for h in range(Hkv):
            k, v = t["k_cache"][b, h, :T + 1].double(), t["v_cache"][b, h, :T + 1].double()
            s = (t["q"][b, h * G:(h + 1) * G].double() @ k.t()) * scale
            lse[b, h * G:(h + 1) * G] = torch.logsumexp(s, 1)
            o[b, h * G:(h + 1) * G] = torch.softmax(s, 1) @ v
    return o, lse, t["k_cache"].double(), t["v_cache"].double()
