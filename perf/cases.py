"""The calls that are timed: what a program using this library has it do, over the sizes it meets.

A program folds each weight once when a model is loaded and then calls the fused ops: few rows per
call while it decodes (one row per running sequence), some tens to some hundreds when it batches
sequences or cuts prompts into chunks, thousands in a prefill.  ``listed()`` gives the cases,
``draw()`` more of the same ranges; ``prepare()`` makes what the program holds before a call and
``run()`` is the call.
"""
from __future__ import annotations

import math

import torch

from paper_2407_09577_amd import flashnorm as fn

EPS = 1e-6
Q_SCALE = 0.125
SEQ = 2048          # tokens per sequence: positions run 0 .. SEQ - 1
KINDS = ("linear", "glu", "rope", "layernorm")


def listed():
    return [
        # One sequence decoding: the FFN input projection of a Llama-7B layer, the largest weight stream of a token.
        {"name": "decode_glu_m1", "kind": "glu", "dtype": "bf16", "M": 1, "K": 4096, "N": 11008},
        # A few sequences decoding: the fused QKV projection with RoPE of a grouped-query layer (32 + 8 + 8 heads).
        {"name": "decode_rope_m7", "kind": "rope", "dtype": "bf16", "M": 7, "K": 4096, "Hq": 32, "Hkv": 8, "h": 128},
        # Batched serving: 64 sequences decode together through the same FFN input projection.
        {"name": "batch_glu_m64", "kind": "glu", "dtype": "bf16", "M": 64, "K": 4096, "N": 11008},
        # A ragged chunk of a prompt through the Llama-7B QKV projection with RoPE.
        {"name": "chunk_rope_m333", "kind": "rope", "dtype": "bf16", "M": 333, "K": 4096, "Hq": 32, "Hkv": 32, "h": 128},
        # A small model's prefill (SmolLM2-135M width).
        {"name": "prefill_smollm2", "kind": "linear", "dtype": "bf16", "M": 2048, "K": 576, "N": 1536},
        # A large model's prefill: the Llama-7B QKV projection, the benchmark's default workload.
        {"name": "prefill_llama7b_qkv", "kind": "linear", "dtype": "bf16", "M": 4096, "K": 4096, "N": 12288},
        # A prefill's FFN input projection at Llama-7B width, the largest share of its arithmetic.
        {"name": "prefill_glu_m2048", "kind": "glu", "dtype": "bf16", "M": 2048, "K": 4096, "N": 11008},
        # A LayerNorm model's projection in prefill.
        {"name": "prefill_layernorm", "kind": "layernorm", "dtype": "bf16", "M": 4096, "K": 4096, "N": 4096},
        # The MLA down-projection with its latent norm and rotary key: a narrow output over a long K.
        {"name": "prefill_mla", "kind": "mla", "dtype": "bf16", "M": 4096, "K": 5120, "L": 512, "R": 64},
        # The smallest call: sixteen rows in fp32, where latency counts.
        {"name": "tiny_fp32", "kind": "linear", "dtype": "f32", "M": 16, "K": 576, "N": 576},
        # An fp32 model's prefill.
        {"name": "prefill_fp32", "kind": "linear", "dtype": "f32", "M": 500, "K": 2048, "N": 2048},
        # Loading a model: a LayerNorm layer's [N, K] weight folded with its g and beta (with the sums that the call needs).
        {"name": "load_fold", "kind": "fold", "dtype": "bf16", "K": 4096, "N": 4096, "beta": True, "transposed": True},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def _depth(rng, lo, hi, unit):
    """A K of the range: mostly a multiple of 64, else of the unit that the dtype needs."""
    u = 64 if rng.random() < 0.6 else unit
    return max(u, _log(rng, lo, hi) // u * u)


def draw(rng):
    family = rng.choice(("decode", "batch", "prefill", "prefill", "mla", "fp32", "fold"))
    if family == "fold":
        K = _depth(rng, 512, 8192, 8)
        return {"kind": "fold", "dtype": rng.choice(("bf16", "bf16", "f32")), "K": K,
                "N": min(_log(rng, 512, 12288), (1 << 25) // K), "beta": rng.random() < 0.5,
                "transposed": rng.random() < 0.7}
    if family == "mla":
        return {"kind": "mla", "dtype": "bf16", "M": _log(rng, 64, 4096), "K": _depth(rng, 1024, 7168, 8),
                "L": rng.choice((256, 384, 512, 768, 1536)), "R": rng.choice((0, 32, 64, 128))}
    if family == "fp32":
        kind, dtype, M, K = rng.choice(KINDS), "f32", _log(rng, 1, 1024), _depth(rng, 256, 4096, 4)
        most = min(4e9 / (M * K), 8192.0)
    else:
        kind, dtype = rng.choice(KINDS), "bf16"
        M = {"decode": lambda: _log(rng, 1, 16), "batch": lambda: _log(rng, 17, 256),
             "prefill": lambda: _log(rng, 257, 4096)}[family]()
        K = _depth(rng, 512, 8192, 8)
        most = min(2.5e8 / K, 1.8e11 / (M * K) / 2, 20480.0)
    if kind == "rope":
        h = rng.choice((64, 128))
        Hkv, group = rng.choice((4, 8, 16)), rng.choice((1, 2, 4))
        while Hkv > 1 and (group + 2) * Hkv * h > most:
            Hkv //= 2
        Hq = group * Hkv
        return {"kind": kind, "dtype": dtype, "M": M, "K": K, "Hq": Hq, "Hkv": Hkv, "h": h}
    N = _log(rng, min(512.0, most / 2), most)
    if rng.random() < 0.5:
        N = max(64, N // 64 * 64)
    return {"kind": kind, "dtype": dtype, "M": M, "K": K, "N": N // 2 if kind == "glu" else N}


def _width(c):
    """Columns of the logical weight."""
    if c["kind"] == "rope":
        return (c["Hq"] + 2 * c["Hkv"]) * c["h"]
    if c["kind"] == "mla":
        return c["L"] + c["R"]
    return 2 * c["N"] if c["kind"] == "glu" else c["N"]


def _inputs(c, seed):
    """Seeded inputs: activations with 1% outlier rows (LayerNorm: mean 0.5), weights of variance 1/K
    as a linear layer holds them ([N, K]), norm weights around 1."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    dt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32

    def normal(*shape):
        return torch.randn(*shape, generator=gen, device="cuda", dtype=torch.float32)

    K, N = c["K"], _width(c)
    x = {"g": torch.rand(K, generator=gen, device="cuda") + 0.5}
    if c["kind"] == "fold" and not c["transposed"]:
        x["W"] = (normal(K, N) * K ** -0.5).to(dt)
    else:
        x["W"] = (normal(N, K) * K ** -0.5).to(dt).t()
    if c["kind"] == "layernorm" or c.get("beta"):
        x["beta"] = normal(K) * 0.1 ** 0.5
    if c["kind"] == "fold":
        return x
    M = c["M"]
    a = normal(M, K)
    if c["kind"] == "layernorm":
        a += 0.5
    a[torch.randperm(M, generator=gen, device="cuda")[: M // 100]] *= 20.0
    x["a"] = a.to(dt)
    half = c["h"] // 2 if c["kind"] == "rope" else c["R"] // 2 if c["kind"] == "mla" else 0
    if half:
        x["pos"] = ((torch.arange(M, device="cuda") + seed) % SEQ).to(torch.int32)
        ang = (torch.arange(SEQ, dtype=torch.float64, device="cuda")[:, None]
               * 10000.0 ** (-torch.arange(half, dtype=torch.float64, device="cuda") / half))
        x["cos"], x["sin"] = ang.cos().float(), ang.sin().float()
    if c["kind"] == "mla":
        x["g_lat"] = torch.rand(c["L"], generator=gen, device="cuda") + 0.5
    return x


def prepare(case, seed):
    x = _inputs(case, seed)
    if case["kind"] == "fold":
        return case, x, None
    glu, ln = case["kind"] == "glu", case["kind"] == "layernorm"
    packed = fn.fold_weights(x["W"], x["g"], beta=x.get("beta"),
                             layout=fn.FN_LAYOUT_GLU if glu else fn.FN_LAYOUT_LINEAR, colsum=ln, c_star=ln)
    del x["W"]  # the program keeps the packed weight
    return case, x, packed


def run(state):
    c, x, packed = state
    kind = c["kind"]
    if kind == "fold":
        ln = c["beta"]
        Ws, colsum, c_star = fn.fold_weights(x["W"], x["g"], beta=x.get("beta"), colsum=ln, c_star=ln)
        return {"W_star": Ws, "colsum": colsum, "c_star": c_star}
    Ws, colsum, c_star = packed
    if kind == "linear":
        return fn.flashnorm_linear(x["a"], Ws, c["N"], EPS)
    if kind == "glu":
        return fn.flashnorm_glu(x["a"], Ws, c["N"], EPS)
    if kind == "layernorm":
        return fn.flashnorm_layernorm_linear(x["a"], Ws, colsum, c_star, c["N"], EPS)
    if kind == "rope":
        return fn.flashnorm_qkv_rope(x["a"], Ws, c["Hq"], c["Hkv"], c["h"], EPS, x["pos"], x["cos"], x["sin"], Q_SCALE)
    return fn.flashnorm_mla_latent(x["a"], Ws, c["L"], c["R"], x["g_lat"], EPS, EPS, positions=x.get("pos"),
                                   cos_tab=x.get("cos"), sin_tab=x.get("sin"))


def work(case):
    size = 2 if case["dtype"] == "bf16" else 4
    K, N = case["K"], _width(case)
    if case["kind"] == "fold":
        return {"bytes": 2 * K * N * size + 4 * K + (4 * K + 8 * N if case["beta"] else 0),
                "flops": K * N * (4 if case["beta"] else 1)}
    M, out = case["M"], case["N"] if case["kind"] == "glu" else N
    return {"bytes": size * (M * K + K * N + M * out), "flops": 2.0 * M * K * N}


def tolerance(case):
    if case["kind"] == "fold":
        # the packed weight is bytes; the sums are rounded once from 64 bits
        return {"rel": 1e-6, "max": 1e-6, "differ": 0.0}
    if case["dtype"] == "f32":
        return {"rel": 4e-6, "max": 1e-4}
    # bf16: W* and the output are rounded to 8 bits; against 64 bits the paths are 2.4e-3 to 4.5e-3 off
    return {"rel": 1e-2, "max": 0.1}


def exact(case, seed):
    x = {k: v.double() for k, v in _inputs(case, seed).items()}
    W = x["W"]
    if case["kind"] == "fold":
        if not case["beta"]:
            return None  # bytes alone
        stored = x["g"][:, None] * W  # exact in 64 bits, then rounded once to the stored type
        if case["dtype"] == "bf16":
            bits = stored.view(torch.int64)
            stored = ((bits + ((1 << 44) - 1) + ((bits >> 45) & 1)) & -(1 << 45)).view(torch.float64)
        else:
            stored = stored.float().double()
        return {"W_star": None, "colsum": stored.sum(0), "c_star": x["beta"] @ W}
    a, K = x["a"], case["K"]
    if case["kind"] == "layernorm":
        d = a - a.mean(1, keepdim=True)
        return (d / (d.square().mean(1, keepdim=True) + EPS).sqrt() * x["g"] + x["beta"]) @ W
    s = (EPS + a.square().sum(1, keepdim=True) / K).rsqrt()
    t = (a * x["g"]) @ W
    if case["kind"] == "linear":
        return t * s
    if case["kind"] == "glu":
        gate, up = (t * s).chunk(2, dim=1)
        return gate * torch.sigmoid(gate) * up

    def rotate(v, h):
        p = v.reshape(v.shape[0], -1, h // 2, 2)
        at = x["pos"].long()
        co, si = x["cos"][at][:, None], x["sin"][at][:, None]
        return torch.stack((p[..., 0] * co - p[..., 1] * si, p[..., 0] * si + p[..., 1] * co), dim=-1).flatten(1)

    if case["kind"] == "rope":
        q, k, v = (t * s).split([case["Hq"] * case["h"], case["Hkv"] * case["h"], case["Hkv"] * case["h"]], dim=1)
        return torch.cat((rotate(q, case["h"]) * Q_SCALE, rotate(k, case["h"]), v), dim=1)
    lat, key = t.split([case["L"], case["R"]], dim=1)
    lat = lat / (EPS + lat.square().mean(1, keepdim=True)).sqrt() * x["g_lat"]
    return torch.cat((lat, rotate(key * s, case["R"])), dim=1) if case["R"] else lat
