"""Performance cases of the library: what a program that serves a quantised language model has it do, through the public
entry points and at the call rate of such a program (plain calls on the current stream, nothing captured).

    listed()              the named cases
    draw(rng)             one more case of the same ranges (rng: random.Random)
    prepare(case, seed)   packed weights, caches, inputs and output buffers: what the program holds before the call
    run(state)            one pass
    work(case)            bytes and operations that one pass cannot do without
    tolerance(case)       how far another correct implementation of the same precision may be off

Five kinds of work (case["kind"]):

    gemm     one linear layer: Y = X * dequant(W), optionally with the fused bias / residual / silu(gate)*up
    moe      the gated MLP of a mixture-of-experts layer: rows sorted by expert, gate/up call, down call
    decode   one decoding step of an attention layer: store the new token's key and value, attend over the cache
    prompt   one chunk of prompt tokens of an attention layer: store the chunk, attend causally over the cache
    layer    one decoding step through whole transformer layers (four GEMMs, store, attention per layer)

Weights are Gaussian matrices under the group-wise recipe of the 4-bit and 8-bit formats (scale = range / levels rounded to
fp16, zero-point, clamp), activations, queries, keys and values are Gaussian fp16.
"""
from __future__ import annotations

import math

import torch

import paper_2508_15601_amd as tm

HEAD = 128                       # head dimension of the attention entry points
ROOT = HEAD ** -0.5              # softmax scale
BITS = {"int4": 4, "int8": 8, "fp8": 8}
LARGEST_FLOPS = 2.0 * 4096 * 8192 * 28672


def listed():
    return [
        # One sequence being generated: the attention output projection of a 4096-wide model, the smallest call there is.
        {"name": "gemm_int4_4096x4096_m1", "kind": "gemm", "format": "int4", "M": 1, "K": 4096, "N": 4096, "group": 128, "epilogue": "none"},
        # Sixteen sequences being generated: fused gate+up projection with its activation.
        {"name": "gemm_int4_gate_up_m16", "kind": "gemm", "format": "int4", "M": 16, "K": 4096, "N": 22016, "group": 128, "epilogue": "silu_mul"},
        # A busier server, an odd number of sequences: down projection with the residual add.
        {"name": "gemm_int4_down_m50", "kind": "gemm", "format": "int4", "M": 50, "K": 11008, "N": 4096, "group": 128, "epilogue": "residual"},
        # A short prompt, or a large decoding batch: a square layer with the finer groups.
        {"name": "gemm_int4_8192x8192_m200", "kind": "gemm", "format": "int4", "M": 200, "K": 8192, "N": 8192, "group": 64, "epilogue": "none"},
        # A long prompt (or several): the MLP of a 70B model, the largest call.
        {"name": "gemm_int4_8192x28672_m4096", "kind": "gemm", "format": "int4", "M": 4096, "K": 8192, "N": 28672, "group": 128, "epilogue": "none"},
        # 8-bit weights, a prompt of ordinary length: FP8 codes with a bias.
        {"name": "gemm_fp8_4096x12288_m700", "kind": "gemm", "format": "fp8", "M": 700, "K": 4096, "N": 12288, "group": 128, "epilogue": "bias"},
        # Decoding with many small experts, eight per token.
        {"name": "moe_128x8_16_tokens", "kind": "moe", "experts": 128, "top_k": 8, "tokens": 16, "hidden": 4096, "inter": 1536},
        # A prompt through few large experts, two per token.
        {"name": "moe_8x2_1000_tokens", "kind": "moe", "experts": 8, "top_k": 2, "tokens": 1000, "hidden": 4096, "inter": 14336},
        # One sequence at an ordinary context: attention at its smallest.
        {"name": "decode_kv8_1x2048", "kind": "decode", "bits": 8, "batch": 1, "q_heads": 32, "kv_heads": 8, "context": 2048},
        # A full server with long contexts over the 4-bit cache.
        {"name": "decode_kv4_32x8192", "kind": "decode", "bits": 4, "batch": 32, "q_heads": 32, "kv_heads": 8, "context": 8192},
        # A prompt of 4000 tokens.
        {"name": "prompt_kv8_4000", "kind": "prompt", "bits": 8, "batch": 1, "q_heads": 32, "kv_heads": 8, "count": 4000, "past": 0},
        # A decoding step of eight sequences through two layers of a 7B model.
        {"name": "layer_kv8_8x2048", "kind": "layer", "bits": 8, "batch": 8, "heads": 32, "kv_heads": 32, "inter": 11008, "context": 2048, "layers": 2},
    ]


def _log_int(rng, lo, hi):
    """A whole number of [lo, hi], even over the logarithm."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def draw(rng):
    kind = rng.choice(["gemm", "gemm", "gemm", "gemm", "moe", "decode", "decode", "prompt", "layer"])
    if kind == "gemm":
        fmt = rng.choice(["int4", "int4", "int4", "int8", "fp8"])
        case = {"kind": kind, "format": fmt, "M": _log_int(rng, 1, 4096), "K": 128 * _log_int(rng, 8, 224),
                "N": 16 * _log_int(rng, 64, 2048), "group": rng.choice([32, 64, 128, 128, 128]),
                "epilogue": rng.choice(["none", "none", "bias", "residual", "silu_mul"])}
        if case["epilogue"] == "silu_mul":               # gate and up side by side; this activation is packed for 4-bit codes
            case["format"] = "int4"
            case["N"] = max(1024, case["N"] // 32 * 32)
        case["M"] = max(1, min(case["M"], int(LARGEST_FLOPS / (2.0 * case["K"] * case["N"]))))
        return case
    if kind == "moe":
        experts = _log_int(rng, 8, 128)
        top_k = min(experts, rng.choice([1, 2, 4, 8]))
        hidden = 128 * _log_int(rng, 12, 64)
        inter = 128 * min(_log_int(rng, 6, 112), int(1.6e9 / (experts * hidden * 128)))
        tokens = _log_int(rng, 1, 4096)
        tokens = max(1, min(tokens, int(0.6 * LARGEST_FLOPS / (6.0 * top_k * hidden * inter))))
        return {"kind": kind, "experts": experts, "top_k": top_k, "tokens": tokens, "hidden": hidden, "inter": inter}
    kv_heads = rng.choice([1, 2, 4, 8, 8, 32])
    per_kv = rng.choice([1, 4, 5, 7, 8]) if kv_heads < 32 else 1
    heads = {"bits": rng.choice([8, 4]), "q_heads": kv_heads * per_kv, "kv_heads": kv_heads}
    if kind == "decode":
        batch = _log_int(rng, 1, 128)
        context = min(_log_int(rng, 128, 32768), max(128, int(2.2e6 / (batch * kv_heads))))
        return {"kind": kind, "batch": batch, "context": context, **heads}
    if kind == "prompt":
        batch = rng.choice([1, 1, 2, 4, 8])
        count = _log_int(rng, 16, 8192)
        past = rng.choice([0, 0, _log_int(rng, 128, 16384)])
        most = 2.7e11 / (4.0 * HEAD * heads["q_heads"] * batch)              # query-key pairs: the cost of a 8192-token prompt at most
        while count > 16 and count * (past + count / 2.0) > most:
            count, past = max(16, count * 3 // 4), past * 3 // 4
        return {"kind": kind, "batch": batch, "count": count, "past": past, **heads}
    heads = rng.choice([16, 28, 32, 40])
    kv_heads = rng.choice([heads, heads // 4])
    return {"kind": "layer", "bits": rng.choice([8, 4]), "batch": _log_int(rng, 1, 64), "heads": heads, "kv_heads": kv_heads,
            "inter": 128 * _log_int(rng, 40, 144), "context": _log_int(rng, 128, 4096), "layers": 2}


# ------------------------------------------------------------------------------------------------------- inputs

class _Inputs:
    """Everything random of a case, from one seed, on the GPU."""

    def __init__(self, seed):
        self.g = torch.Generator(device="cuda")
        self.g.manual_seed(seed)

    def normal(self, *shape, std=1.0):
        return (torch.randn(shape, generator=self.g, device="cuda") * std).to(torch.float16)

    def codes(self, fmt, K, N, group, std):
        """Gaussian [K][N] under the recipe of the format -> (packed words, scales, zeros or None)."""
        words, scales, zeros = [], [], []
        rows = max(group, (1 << 26) // N // group * group)                   # in slices of K: the fp32 matrix stays small
        for k0 in range(0, K, rows):
            r = min(rows, K - k0)
            w = torch.randn((r // group, group, N), generator=self.g, device="cuda") * std
            if fmt == "fp8":
                s = (w.abs().amax(1) / 448.0).to(torch.float16)
                c = (w / s.float()[:, None]).clamp_(-448.0, 448.0).reshape(r, N).to(torch.float8_e4m3fn)
                words.append(c.view(torch.int32))
            else:
                top = 2 ** BITS[fmt] - 1
                mn = w.amin(1)
                s = ((w.amax(1) - mn) / top).to(torch.float16)
                z = (-mn / s.float()).round_().clamp_(0, top)
                c = ((w / s.float()[:, None]).round_() + z[:, None]).clamp_(0, top).reshape(r, N).to(torch.uint8)
                if fmt == "int4":                        # nibble t of a word is column 8j + t
                    c = c[:, 0::2] | (c[:, 1::2] << 4)
                words.append(c.contiguous().view(torch.int32))
                zeros.append(z.to(torch.float16))
            scales.append(s)
        return torch.cat(words), torch.cat(scales), torch.cat(zeros) if zeros else None

    def weight(self, fmt, K, N, group=128, gate_up=False, std=0.02):
        q, s, z = self.codes(fmt, K, N, group, std)
        if gate_up:
            return tm.tm_pack_w4_gate_up(q, s, z, K, N, group)
        if fmt == "fp8":
            return tm.tm_pack_w8_fp8(q, s, K, N, group)
        return (tm.tm_pack_w4 if fmt == "int4" else tm.tm_pack_w8)(q, s, z, K, N, group)

    def cache(self, batch, kv_heads, capacity, bits):
        """A cache whose every token has been stored once (slice by slice)."""
        cache = tm.tm_kv_create(batch, kv_heads, capacity, bits)
        step = max(32, min(cache.capacity, (1 << 26) // (batch * kv_heads * HEAD) // 32 * 32))
        for t in range(0, cache.capacity, step):
            n = min(step, cache.capacity - t)
            at = torch.full((batch,), t, dtype=torch.int32, device="cuda")
            tm.tm_kv_append(cache, self.normal(batch, n, kv_heads, HEAD), self.normal(batch, n, kv_heads, HEAD), at)
        return cache

    def lens(self, batch, context):
        """Tokens cached per sequence: between half the context and all of it, the first sequence's the longest."""
        lens = torch.randint((context + 1) // 2, context + 1, (batch,), generator=self.g, device="cuda", dtype=torch.int32)
        lens[0] = context
        return lens


class _Device:
    """A buffer of a cache as the array interface describes it.  A tensor made from it holds this object and with it the
    cache, whose memory is freed with the last of them."""

    def __init__(self, cache, ptr, nbytes):
        self.cache = cache
        self.__cuda_array_interface__ = {"shape": (nbytes,), "typestr": "|u1", "data": (ptr, False), "version": 3}


def _cache_state(cache):
    """The cache's own buffers, as tensors: the state that storing new tokens updates."""
    k, v, pairs, code_bytes, pair_bytes = tm.tm_kv_raw(cache)
    return [torch.as_tensor(_Device(cache, p, n), device="cuda") for p, n in ((k, code_bytes), (v, code_bytes), (pairs, pair_bytes))]


def _empty(*shape):
    return torch.empty(shape, dtype=torch.float16, device="cuda")


def prepare(case, seed):
    r = _Inputs(seed)
    return {"case": case, **globals()["_prepare_" + case["kind"]](case, r)}


def run(state):
    return globals()["_run_" + state["case"]["kind"]](state)


# --------------------------------------------------------------------------------------------------------- gemm

def _prepare_gemm(c, r):
    M, K, N, epi = c["M"], c["K"], c["N"], c["epilogue"]
    s = {"W": r.weight(c["format"], K, N, c["group"], gate_up=epi == "silu_mul"), "X": r.normal(M, K),
         "Y": _empty(M, N // 2 if epi == "silu_mul" else N)}
    if epi == "bias":
        s["bias"] = r.normal(N)
    if epi == "residual":
        s["residual"] = r.normal(M, N)
    return s


def _run_gemm(s):
    epi = s["case"]["epilogue"]
    if epi == "none":
        return tm.tm_gemm_w4a16(s["X"], s["W"], s["Y"])
    if epi == "silu_mul":
        return tm.tm_gemm_w4a16_ex(s["X"], s["W"], s["Y"], act=tm.TM_ACT_SILU_MUL)
    return tm.tm_gemm_w4a16_ex(s["X"], s["W"], s["Y"], bias=s.get("bias"), residual=s.get("residual"))


def _gemm_work(M, K, N, group, fmt, epilogue):
    out = N // 2 if epilogue == "silu_mul" else N
    more = {"none": 0, "silu_mul": 0, "bias": 2 * N, "residual": 2 * M * N}[epilogue]
    pairs = (2 if fmt == "fp8" else 4) * K * N // group
    return K * N * BITS[fmt] // 8 + pairs + 2 * M * K + 2 * M * out + more, 2.0 * M * K * N


# ---------------------------------------------------------------------------------------------------------- moe

def _prepare_moe(c, r):
    E, H, I, rows = c["experts"], c["hidden"], c["inter"], c["tokens"] * c["top_k"]
    up = [r.weight("int4", H, 2 * I, gate_up=True) for _ in range(E)]
    down = [r.weight("int4", I, H) for _ in range(E)]
    # every token goes to top_k different experts, all equally likely
    picks = torch.rand((c["tokens"], E), generator=r.g, device="cuda").topk(c["top_k"], dim=1).indices
    offsets = torch.zeros(E + 1, dtype=torch.int32, device="cuda")
    offsets[1:] = torch.bincount(picks.flatten(), minlength=E).cumsum(0)
    return {"up": tm.tm_group_experts(up), "down": tm.tm_group_experts(down), "offsets": offsets,
            "X": r.normal(rows, H), "A": _empty(rows, I), "Y": _empty(rows, H)}


def _run_moe(s):
    tm.tm_gemm_w4a16_grouped_act(s["X"], s["up"], s["offsets"], s["A"], act=tm.TM_ACT_SILU_MUL)
    tm.tm_gemm_w4a16_grouped(s["A"], s["down"], s["offsets"], s["Y"])
    return s["A"], s["Y"]


# ------------------------------------------------------------------------------------------------------- decode

def _prepare_decode(c, r):
    B, Hq, Hk, T = c["batch"], c["q_heads"], c["kv_heads"], c["context"]
    cache, lens = r.cache(B, Hk, T, c["bits"]), r.lens(B, T)
    return {"cache": cache, "held": _cache_state(cache), "lens": lens, "at": lens - 1, "Q": r.normal(B, Hq, HEAD),
            "K": r.normal(B, 1, Hk, HEAD), "V": r.normal(B, 1, Hk, HEAD), "O": _empty(B, Hq, HEAD)}


def _run_decode(s):
    tm.tm_kv_append(s["cache"], s["K"], s["V"], s["at"])
    tm.tm_attn_decode(s["Q"], s["cache"], s["lens"], s["O"], ROOT, max_len=s["case"]["context"])
    return [s["O"]] + s["held"]


def _token_bytes(bits):
    """Codes and scale/zero pairs of one token and KV head, key and value."""
    return 2 * HEAD * bits // 8 + 8


def _decode_work(B, Hq, Hk, T, bits):
    tokens = B * 0.75 * T                                # lens: half to all of the context
    return Hk * (tokens * _token_bytes(bits) + B * 4 * HEAD) + 4 * B * Hq * HEAD, 4.0 * tokens * Hq * HEAD


# ------------------------------------------------------------------------------------------------------- prompt

def _prepare_prompt(c, r):
    B, Hq, Hk, n, past = c["batch"], c["q_heads"], c["kv_heads"], c["count"], c["past"]
    cache = r.cache(B, Hk, past + n, c["bits"])
    return {"cache": cache, "held": _cache_state(cache), "at": torch.full((B,), past, dtype=torch.int32, device="cuda"),
            "Q": r.normal(B, n, Hq, HEAD), "K": r.normal(B, n, Hk, HEAD), "V": r.normal(B, n, Hk, HEAD), "O": _empty(B, n, Hq, HEAD)}


def _run_prompt(s):
    tm.tm_kv_append(s["cache"], s["K"], s["V"], s["at"])
    tm.tm_attn_prefill(s["Q"], s["cache"], s["at"], s["O"], ROOT)
    return [s["O"]] + s["held"]


# -------------------------------------------------------------------------------------------------------- layer

def _layer_shapes(c):
    """The four linear layers: (name, K, N, epilogue)."""
    hidden, qkv = c["heads"] * HEAD, (c["heads"] + 2 * c["kv_heads"]) * HEAD
    return [("qkv", hidden, qkv, "none"), ("out", hidden, hidden, "residual"), ("up", hidden, 2 * c["inter"], "silu_mul"),
            ("down", c["inter"], hidden, "residual")]


def _prepare_layer(c, r):
    B, Hq, Hk, T = c["batch"], c["heads"], c["kv_heads"], c["context"]
    stack = []
    for _ in range(c["layers"]):
        # the spread keeps activations of every layer near one without the norms between them
        w = {name: r.weight("int4", K, N, gate_up=epi == "silu_mul", std=K ** -0.5) for name, K, N, epi in _layer_shapes(c)}
        w["cache"] = r.cache(B, Hk, T, c["bits"])
        w["held"] = _cache_state(w["cache"])
        w["y"] = _empty(B, Hq * HEAD)
        stack.append(w)
    lens, hidden = r.lens(B, T), Hq * HEAD
    return {"stack": stack, "lens": lens, "at": lens - 1, "x": r.normal(B, hidden), "qkv": _empty(B, (Hq + 2 * Hk) * HEAD),
            "att": _empty(B, Hq, HEAD), "mid": _empty(B, hidden), "act": _empty(B, c["inter"])}


def _run_layer(s):
    c = s["case"]
    B, Hq, Hk = c["batch"], c["heads"], c["kv_heads"]
    x, mid, act, att = s["x"], s["mid"], s["act"], s["att"]
    for w in s["stack"]:
        qkv = tm.tm_gemm_w4a16(x, w["qkv"], s["qkv"])
        q, k, v = (t.contiguous() for t in qkv.split((Hq * HEAD, Hk * HEAD, Hk * HEAD), dim=1))
        tm.tm_kv_append(w["cache"], k.view(B, 1, Hk, HEAD), v.view(B, 1, Hk, HEAD), s["at"])
        tm.tm_attn_decode(q.view(B, Hq, HEAD), w["cache"], s["lens"], att, ROOT, max_len=c["context"])
        tm.tm_gemm_w4a16_ex(att.view(B, Hq * HEAD), w["out"], mid, residual=x)
        tm.tm_gemm_w4a16_ex(mid, w["up"], act, act=tm.TM_ACT_SILU_MUL)
        x = tm.tm_gemm_w4a16_ex(act, w["down"], w["y"], residual=mid)
    return [[w["y"]] + w["held"] for w in s["stack"]]


# ---------------------------------------------------------------------------------------------- work and tolerance

def work(case):
    c, kind = case, case["kind"]
    if kind == "gemm":
        b, f = _gemm_work(c["M"], c["K"], c["N"], c["group"], c["format"], c["epilogue"])
    elif kind == "moe":
        E, H, I, rows = c["experts"], c["hidden"], c["inter"], c["tokens"] * c["top_k"]
        busy = E * (1.0 - (1.0 - c["top_k"] / E) ** c["tokens"])             # experts that get a row, on average
        b = busy * 3 * H * I * (0.5 + 4 / 128) + 2 * rows * (2 * H + 2 * I)
        f = 6.0 * rows * H * I
    elif kind == "decode":
        b, f = _decode_work(c["batch"], c["q_heads"], c["kv_heads"], c["context"], c["bits"])
    elif kind == "prompt":
        B, Hq, Hk, n, past = c["batch"], c["q_heads"], c["kv_heads"], c["count"], c["past"]
        b = B * (Hk * (n * 4 * HEAD + (past + n) * _token_bytes(c["bits"])) + 4 * n * Hq * HEAD)
        f = 4.0 * B * Hq * HEAD * (n * past + n * (n + 1) / 2.0)
    else:
        parts = [_gemm_work(c["batch"], K, N, 128, "int4", epi) for _, K, N, epi in _layer_shapes(c)]
        parts.append(_decode_work(c["batch"], c["heads"], c["kv_heads"], c["context"], c["bits"]))
        b, f = (c["layers"] * sum(p[i] for p in parts) for i in (0, 1))
    return {"bytes": b, "flops": f}


def tolerance(case):
    """One product: fp16 result (2^-11 of a value at most) of fp16 factors, of which (q - z) * s may be rounded to fp16
    (again 2^-11) or not.  The gated activation multiplies two such results, a chain of layers adds up its stages.
    Attention rounds the probabilities and the result to fp16.  Stored codes follow from the inputs alone, bit for bit, except
    where an earlier stage of the same pass computes the keys and values: there a rounding tie may move a code by one."""
    kind = case["kind"]
    if kind == "layer":
        return {"rel": 6e-3, "max": 6e-2, "differ": 2e-3}
    if kind == "moe" or case.get("epilogue") == "silu_mul":
        return {"rel": 4e-3, "max": 4e-2}
    return {"rel": 2e-3, "max": 2e-2}
