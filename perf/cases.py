"""What a user of this library runs, as cases that can be timed and checked.

The library is one linear layer (activations fp16 or bf16, weights in 4 or 8
bits) in its two forms, the decode GEMV and the prefill GEMM, the gated MLP
built of them, and the packing that a weight goes through when a model is
loaded.  The shapes are the linear layers that the repository's own workloads
and the paper name: Llama-3-8B (hidden 4096, MLP 14336), the 2048-wide models
(Gemma-2B, Qwen2.5-3B), their tensor-parallel shards, and the 32K dimensions of
the prompt-length sweep.  A state holds what a serving program holds: the
packed weights and the activations, on the GPU.
"""
from __future__ import annotations

import math

import torch

from paper_2606_11357_amd import tilefuse as tf

_SCALES = {4: (0.005, 0.02), 8: (0.0003, 0.001)}     # the ranges of the repository's workloads


def _case(name, kind, bits, dtype, M, K, N, group=128):
    c = {"kind": kind, "bits": bits, "dtype": dtype, "M": M, "K": K, "N": N, "group": group}
    return {"name": name, **c} if name else c


def listed():
    return [
        # one token of one sequence through the up (or gate) projection of the MLP: most of what generation does
        _case("decode_w4_m1", "gemv", 4, "fp16", 1, 4096, 14336),
        # the same token through an 8-bit attention output projection: the smallest call, bound by latency
        _case("decode_w8_m1_bf16", "gemv", 8, "bf16", 1, 4096, 4096),
        # eight sequences decoded together (or eight speculated tokens) through the decode entry point
        _case("decode_w4_m8_bf16", "gemv", 4, "bf16", 8, 4096, 14336),
        # sixteen rows of a 2048-wide model's attention projection: a small batch through the GEMM entry point
        _case("gemm_w4_m16", "gemm", 4, "fp16", 16, 2048, 2048),
        # continuous batching with an odd number of sequences
        _case("gemm_w4_m49_bf16", "gemm", 4, "bf16", 49, 4096, 14336),
        # a short prompt through the down projection (long K, few columns)
        _case("gemm_w4_m200_down", "gemm", 4, "fp16", 200, 14336, 4096),
        # a chunk of a chunked prefill through an 8-bit attention projection
        _case("gemm_w8_m512", "gemm", 8, "fp16", 512, 4096, 4096),
        # a row-parallel shard of an 11008-wide MLP over eight devices (11008 / 8 = 1376 rows, groups of 32)
        _case("gemm_w4_m333_shard", "gemm", 4, "fp16", 333, 1376, 2048, 32),
        # the gated MLP of one layer over a ragged prompt: gate and up, activation, down
        _case("mlp_w4_m1000_bf16", "mlp", 4, "bf16", 1000, 4096, 14336),
        # a prompt of 2048 tokens through the down projection
        _case("gemm_w4_m2048_down", "gemm", 4, "fp16", 2048, 14336, 4096),
        # the longest prompt of the sweep through the up projection
        _case("gemm_w4_m8192", "gemm", 4, "fp16", 8192, 4096, 14336),
        # loading a model: one AWQ weight into the library's layout
        _case("pack_w4", "pack", 4, "fp16", 0, 4096, 14336),
    ]


# (K, N) of the linear layers meant above: MLP and attention projections
_LAYERS = [(4096, 14336), (14336, 4096), (4096, 4096), (4096, 1024), (4096, 6144), (4096, 28672),
           (2048, 16384), (16384, 2048), (2048, 11008), (11008, 2048), (2048, 2048), (2048, 256),
           (4096, 1792), (1792, 4096), (4096, 32768), (32768, 8192)]
_MOST_FLOPS = 2 * 8192 * 4096 * 14336


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case: any kind, width and type, over the whole range of rows, on
    a layer named above or on one of any size, with the group sizes in use."""
    kind = rng.choice(["gemv"] * 3 + ["gemm"] * 5 + ["mlp", "pack"])
    bits = rng.choice([4, 4, 8])
    dtype = rng.choice(["fp16", "bf16"])
    group = rng.choice([128] * 5 + [64, 32, 256])
    layers = [kn for kn in _LAYERS if kn[0] % group == 0]
    if kind == "mlp":
        K, N = rng.choice([(4096, 14336), (2048, 11008), (2048, 16384), (4096, 1792)])
        group = min(group, 128)
    elif rng.random() < 0.6:
        K, N = rng.choice(layers)
    else:
        # any layer: K a whole number of groups, N a multiple of 8
        group = rng.choice([128, 128, 64, 32, 96])
        K = group * max(1, _log_int(rng, 512, 12288) // group)
        N = 8 * _log_int(rng, 64, 2048)
    M = {"gemv": rng.randint(1, 8), "gemm": _log_int(rng, 9, 8192), "mlp": _log_int(rng, 1, 4096), "pack": 0}[kind]
    if M:
        per_row = (6 if kind == "mlp" else 2) * K * N
        M = max(1, min(M, _MOST_FLOPS // per_row))
        if K % 128:                       # layers off the usual grid are small ones
            M = max(1, min(M, _MOST_FLOPS // (16 * per_row)))
    return _case("", kind, bits, dtype, M, K, N, group)


def _dt(case):
    return torch.float16 if case["dtype"] == "fp16" else torch.bfloat16


def _weight(case, gen, K, N):
    """One quantized weight as a checkpoint has it (AWQ words, or bytes)."""
    bits, group = case["bits"], case["group"]
    dev = "cuda"
    lo, hi = _SCALES[bits]
    if bits == 4:
        w = {"q": torch.randint(-2 ** 31, 2 ** 31, (K, N // 8), dtype=torch.int32, device=dev, generator=gen),
             "z": torch.randint(-2 ** 31, 2 ** 31, (K // group, N // 8), dtype=torch.int32, device=dev, generator=gen)}
    else:
        w = {"q": torch.randint(0, 256, (K, N), dtype=torch.uint8, device=dev, generator=gen),
             "z": torch.randint(0, 256, (K // group, N), dtype=torch.uint8, device=dev, generator=gen)}
    w["s"] = (lo + (hi - lo) * torch.rand((K // group, N), device=dev, generator=gen)).to(_dt(case))
    return w


def _inputs(case, seed):
    """Activations and weights, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    M, K, N = case["M"], case["K"], case["N"]
    x = torch.randn((M, K), device="cuda", generator=gen).to(_dt(case)) if M else None
    if case["kind"] == "mlp":
        return x, [_weight(case, gen, K, 2 * N), _weight(case, gen, N, K)]
    return x, [_weight(case, gen, K, N)]


def _shapes(case):
    K, N = case["K"], case["N"]
    return [(K, 2 * N), (N, K)] if case["kind"] == "mlp" else [(K, N)]


def prepare(case, seed):
    x, weights = _inputs(case, seed)
    bits, group = case["bits"], case["group"]
    pack = tf.pack_w4 if bits == 4 else tf.pack_w8
    state = {"case": case, "x": x}
    if case["kind"] == "pack":
        # the checkpoint's tensors and the buffer they are packed into
        K, N = case["K"], case["N"]
        state["weight"] = weights[0]
        state["out"] = torch.zeros(tf.packed_bytes(bits, K, N, group), dtype=torch.uint8, device="cuda")
    else:
        state["packed"] = [pack(w["q"], w["z"], w["s"], K, N, group) for w, (K, N) in zip(weights, _shapes(case))]
    return state


_GEMV = {4: tf.w4a16_gemv, 8: tf.w8a16_gemv}
_GEMM = {4: tf.w4a16_gemm, 8: tf.w8a16_gemm}


def run(state):
    case = state["case"]
    kind, bits, K, N, group = case["kind"], case["bits"], case["K"], case["N"], case["group"]
    if kind == "pack":
        w = state["weight"]
        return (tf.pack_w4 if bits == 4 else tf.pack_w8)(w["q"], w["z"], w["s"], K, N, group, out=state["out"])
    x, packed = state["x"], state["packed"]
    if kind == "gemv":
        return _GEMV[bits](x, packed[0], K, N, group)
    if kind == "gemm":
        return _GEMM[bits](x, packed[0], K, N, group)
    f = _GEMV[bits] if case["M"] == 1 else _GEMM[bits]
    gu = f(x, packed[0], K, 2 * N, group)
    return f(tf.silu_mul(gu), packed[1], N, K, group)


def work(case):
    M, group, bits = case["M"], case["group"], case["bits"]
    weights = sum(K * N * bits // 8 + (K // group) * N * (2 + bits / 8) for K, N in _shapes(case))
    if case["kind"] == "pack":
        K, N = case["K"], case["N"]
        # read as they come, written with one byte a zero-point
        return {"bytes": weights + K * N * bits // 8 + (K // group) * N * 3, "flops": 0}
    flops = sum(2 * M * K * N for K, N in _shapes(case))
    ends = case["K"] + (case["K"] if case["kind"] == "mlp" else case["N"])
    return {"bytes": weights + 2 * M * ends, "flops": flops}


def tolerance(case):
    if case["kind"] == "pack":
        return "exact"
    # Measured against exact(): fp16 2 to 3e-4, bf16 1.7 to 2.4e-3 (the output's own rounding, and in the tiled
    # GEMMs each weight's), a whole MLP three roundings more; four times that.
    rel = 1.2e-3 if case["dtype"] == "fp16" else 1e-2
    return {"rel": 2 * rel if case["kind"] == "mlp" else rel}


def _nibbles(words, N):
    shift = torch.arange(0, 32, 4, device=words.device, dtype=torch.int32)
    return ((words[:, :, None] >> shift) & 15).reshape(words.shape[0], N)


def _dequant64(case, w, N):
    q, z = (_nibbles(w["q"], N), _nibbles(w["z"], N)) if case["bits"] == 4 else (w["q"], w["z"])
    rep = lambda t: t.double().repeat_interleave(case["group"], 0)  # noqa: E731
    return q.double().sub_(rep(z)).mul_(rep(w["s"]))


def exact(case, seed):
    if case["kind"] == "pack":
        return None
    x, weights = _inputs(case, seed)
    y = x.double()
    for i, (w, (K, N)) in enumerate(zip(weights, _shapes(case))):
        y = y @ _dequant64(case, w, N)
        if case["kind"] == "mlp" and i == 0:
            g, u = y[:, :N // 2], y[:, N // 2:]
            y = g / (1 + torch.exp(-g)) * u
    return y
