"""The work this library is measured on: products, a linear layer's training step, a convolution layer and top-k selection.

Every case goes through the public entry points (``gemm_run``, ``gemm_run_ex``, ``conv2d_run``, ``topk_run``) as a
program that links the library does: buffers, descriptors and scratch are made once (``prepare``), a pass launches.
Sizes are those of ``bench.py`` and of ``paper_2605_28213_amd/inputs.py`` where those name one, generic otherwise.
``draw`` gives further cases of the same families over the whole range of sizes, most of them ragged.
"""
import math

import torch

from paper_2605_28213_amd import conv, gemm, topk

K4 = gemm.GEMM_K4_MFMA
ROW, COL = gemm.GEMM_ROW_MAJOR, gemm.GEMM_COL_MAJOR
CODES = {"f32": gemm.GEMM_F32, "bf16": gemm.GEMM_BF16, "f16": gemm.GEMM_F16, "e4m3": gemm.GEMM_FP8_E4M3}
TORCH = {"f32": torch.float32, "bf16": torch.bfloat16, "f16": torch.float16, "e4m3": torch.float8_e4m3fn}
BYTES = {"f32": 4, "bf16": 2, "f16": 2, "e4m3": 1}
OUT = {"f32": "f32", "bf16": "bf16", "f16": "f16", "e4m3": "bf16"}      # the output type gemm_run gives each input type


def listed():
    return [
        # The short form of the call (gemm_run: tight rows, default layouts, no scratch).
        # fp32, the smallest product of the benchmark: a latency, as in a small layer or a solver's inner step.
        {"name": "f32_256", "kind": "short", "dtype": "f32", "M": 256, "N": 256, "K": 256},
        # fp32 of ordinary size: the type a program starts from.
        {"name": "f32_2048", "kind": "short", "dtype": "f32", "M": 2048, "N": 2048, "K": 2048},
        # fp16, both operands row-major as a framework's tensors are: an ordinary size ...
        {"name": "f16_1000", "kind": "short", "dtype": "f16", "M": 1000, "N": 1000, "K": 1000},
        # ... and the benchmark's ragged one, where no row is aligned.
        {"name": "f16_ragged", "kind": "short", "dtype": "f16", "M": 4099, "N": 4093, "K": 4097},
        # The benchmark's headline product: bf16, weight stored [N][K], the largest work here.
        {"name": "bf16_8192", "kind": "short", "dtype": "bf16", "M": 8192, "N": 8192, "K": 8192},
        # One training step of a linear layer in bf16: forward with bias, gradient of the input, gradient of the
        # weight (three layouts of the operands), scratch lent as gemm_query asks for it.
        {"name": "linear_train", "kind": "linear", "dtype": "bf16", "tokens": 4096, "inp": 2048, "out": 2048},
        # Decoding: few rows against a large weight, the benchmark's 16 rows (one wave of requests) and 128 (a full batch).
        {"name": "decode_16", "kind": "decode", "dtype": "bf16", "M": 16, "N": 16384, "K": 16384},
        {"name": "decode_128", "kind": "decode", "dtype": "bf16", "M": 128, "N": 16384, "K": 16384},
        # Quantised inference: the benchmark's batch of e4m3 products with a scale per problem, bf16 out.
        {"name": "e4m3_batched", "kind": "batched", "dtype": "e4m3", "batch": 64, "M": 1024, "N": 1024, "K": 1024},
        # The benchmark's convolution layer.
        {"name": "conv_3x3", "kind": "conv", "dtype": "f16", "n": 8, "hw": 56, "C": 64, "F": 128, "ksize": 3, "stride": 1},
        # Selection: the benchmark's rows (attention scores), and rows as long as a vocabulary (sampling), which the
        # resident state refuses and the streaming one takes.
        {"name": "topk_4096", "kind": "topk", "batch": 64, "n": 4096, "k": 512},
        {"name": "topk_131072", "kind": "topk", "batch": 8, "n": 131072, "k": 64},
    ]


def _log(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["f32", "f16", "bf16", "linear", "decode", "batched", "conv", "topk"])
    if kind == "f32":
        return {"kind": "short", "dtype": "f32", "M": _log(rng, 64, 2300), "N": _log(rng, 64, 2300), "K": _log(rng, 64, 2300)}
    if kind == "f16":
        return {"kind": "short", "dtype": "f16", "M": _log(rng, 128, 4300), "N": _log(rng, 128, 4300), "K": _log(rng, 128, 4300)}
    if kind == "bf16":          # K contiguous in both operands, K of whole 128-byte lines; rows and columns of any number
        return {"kind": "short", "dtype": "bf16", "M": _log(rng, 256, 8000), "N": _log(rng, 256, 8000), "K": 64 * _log(rng, 4, 128)}
    if kind == "linear":        # widths in steps of 8 elements, any number of tokens
        return {"kind": "linear", "dtype": rng.choice(["bf16", "f16"]), "tokens": _log(rng, 128, 6000),
                "inp": 8 * _log(rng, 32, 512), "out": 8 * _log(rng, 32, 512)}
    if kind == "decode":
        return {"kind": "decode", "dtype": rng.choice(["bf16", "f16", "e4m3"]), "M": _log(rng, 1, 128),
                "N": 16 * _log(rng, 64, 1024), "K": 128 * _log(rng, 8, 128)}
    if kind == "batched":
        return {"kind": "batched", "dtype": rng.choice(["e4m3", "bf16"]), "batch": _log(rng, 2, 64), "M": _log(rng, 100, 1030),
                "N": _log(rng, 100, 1030), "K": 128 * rng.randint(1, 8)}
    if kind == "conv":          # first layers (few channels) to deep ones
        return {"kind": "conv", "dtype": rng.choice(["f16", "bf16"]), "n": _log(rng, 1, 16), "hw": rng.choice([7, 13, 14, 28, 55, 56, 112]),
                "C": rng.choice([3, 24, 64, 64, 128, 192, 256]), "F": 8 * _log(rng, 4, 48), "ksize": rng.choice([1, 3, 3, 5]),
                "stride": rng.choice([1, 1, 2])}
    n = _log(rng, 300, 200000)
    return {"kind": "topk", "batch": _log(rng, 1, 128), "n": n, "k": _log(rng, 1, min(2048, n // 2))}


def _randn(shape, dtype, gen, std=1.0):
    x = torch.randn(shape, generator=gen, device="cuda", dtype=torch.float32) * std
    return x.clamp_(-448, 448).to(TORCH[dtype]) if dtype == "e4m3" else x.to(TORCH[dtype])


def _uniform(shape, dtype, gen):
    return (torch.rand(shape, generator=gen, device="cuda", dtype=torch.float32) * 2 - 1).to(TORCH[dtype])


def _empty(shape, dtype):
    return torch.empty(shape, device="cuda", dtype=TORCH[dtype])


def _lend(desc, ptrs):
    """Scratch for a descriptor, as much as the library asks for; returns the buffer (kept by the caller)."""
    need = gemm.gemm_query(K4, desc, *ptrs).workspace_bytes
    if not need:
        return None
    ws = torch.empty(need, dtype=torch.uint8, device="cuda")
    desc.workspace, desc.workspace_bytes = ws.data_ptr(), need
    return ws


def _ok(rc):
    if rc != gemm.GEMM_OK:
        raise RuntimeError(gemm.gemm_status_string(rc))


def prepare(case, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    kind = case["kind"]
    stream = torch.cuda.current_stream()
    if kind == "short":
        dt, M, N, K = case["dtype"], case["M"], case["N"], case["K"]
        if dt == "bf16":        # the weight is [N][K]
            A, B = _randn((M, K), dt, gen, K ** -0.5), _randn((N, K), dt, gen, K ** -0.5)
        else:
            A, B = _uniform((M, K), dt, gen), _uniform((K, N), dt, gen)
        return {"kind": kind, "args": (K4, M, N, K, CODES[dt]), "A": A, "B": B, "C": _empty((M, N), dt)}
    if kind == "linear":
        dt, T, I, O = case["dtype"], case["tokens"], case["inp"], case["out"]
        X, W, dY = _randn((T, I), dt, gen), _randn((O, I), dt, gen, I ** -0.5), _randn((T, O), dt, gen, 0.02)
        bias = torch.randn(O, generator=gen, device="cuda") * 0.1
        Y, dX, dW = _empty((T, O), dt), _empty((T, I), dt), _empty((O, I), dt)
        c = CODES[dt]
        calls = [(gemm.make_desc(T, O, I, c, c, ROW, COL, bias=bias, stream=stream), X, W, Y),      # Y = X W^T + bias
                 (gemm.make_desc(T, I, O, c, c, ROW, ROW, stream=stream), dY, W, dX),               # dX = dY W
                 (gemm.make_desc(O, I, T, c, c, COL, ROW, stream=stream), dY, X, dW)]               # dW = dY^T X
        return {"kind": kind, "calls": calls, "scratch": [_lend(d, p) for d, *p in calls], "bias": bias, "outs": (Y, dX, dW)}
    if kind == "decode":
        dt, M, N, K = case["dtype"], case["M"], case["N"], case["K"]
        std = 1.0 if dt == "e4m3" else 0.02
        A, B, C = _randn((M, K), dt, gen, std), _randn((N, K), dt, gen, std), _empty((M, N), OUT[dt])
        scales = [torch.rand(1, generator=gen, device="cuda") * 1.5 + 0.5 for _ in range(2)] if dt == "e4m3" else [None, None]
        d = gemm.make_desc(M, N, K, CODES[dt], CODES[OUT[dt]], ROW, COL, scale_a=scales[0], scale_b=scales[1], stream=stream)
        return {"kind": kind, "calls": [(d, A, B, C)], "scratch": _lend(d, (A, B, C)), "scales": scales, "outs": C}
    if kind == "batched":
        dt, b, M, N, K = case["dtype"], case["batch"], case["M"], case["N"], case["K"]
        A, B, C = _randn((b, M, K), dt, gen), _randn((b, N, K), dt, gen), _empty((b, M, N), OUT[dt])
        scales = [torch.rand(b, generator=gen, device="cuda") * 1.5 + 0.5 for _ in range(2)] if dt == "e4m3" else [None, None]
        d = gemm.make_desc(M, N, K, CODES[dt], CODES[OUT[dt]], ROW, COL, batch=b, scale_a=scales[0], scale_b=scales[1], stream=stream)
        return {"kind": kind, "calls": [(d, A, B, C)], "scratch": _lend(d, (A, B, C)), "scales": scales, "outs": C}
    if kind == "conv":
        dt, n, hw, C, F, k, s = (case[x] for x in ("dtype", "n", "hw", "C", "F", "ksize", "stride"))
        x, w = _uniform((n, hw, hw, C), dt, gen), _randn((F, k, k, C), dt, gen, (k * k * C) ** -0.5)
        d = conv.make_desc(n, hw, hw, C, F, k, k, CODES[dt], CODES[dt], stride=(s, s), pad=(k // 2, k // 2), stream=stream)
        variant, ws = conv.CONV_C2_IMPLICIT_MFMA, None
        if conv.conv2d_query(variant, d, x, w).status != gemm.GEMM_OK:      # too few channels for the gather: patches are written out
            variant = conv.CONV_C1_IM2COL_MFMA
            ws = torch.empty(conv.conv2d_query(variant, d, x, w).workspace_bytes, dtype=torch.uint8, device="cuda")
            d.workspace, d.workspace_bytes = ws.data_ptr(), ws.numel()
        q = conv.conv2d_query(variant, d, x, w)
        return {"kind": kind, "variant": variant, "desc": d, "scratch": ws, "x": x, "w": w, "y": _empty((n, q.P, q.Q, F), dt)}
    b, n, k = case["batch"], case["n"], case["k"]
    ld = (n + 3) // 4 * 4                                                   # rows padded to 16 bytes
    x = torch.randn((b, ld), generator=gen, device="cuda")
    d = topk.make_desc(b, n, k, ld=ld, stream=stream)
    variant = topk.TOPK_T2_RESIDENT if topk.topk_query(topk.TOPK_T2_RESIDENT, d, x).status == gemm.GEMM_OK else topk.TOPK_T1_RADIX_SELECT
    return {"kind": kind, "variant": variant, "desc": d, "x": x, "idx": torch.empty((b, k), dtype=torch.int32, device="cuda"),
            "val": torch.empty((b, k), device="cuda")}


def run(state):
    kind = state["kind"]
    if kind == "short":
        _ok(gemm.gemm_run(*state["args"], state["A"], state["B"], state["C"]))
        return state["C"]
    if kind == "conv":
        _ok(conv.conv2d_run(state["variant"], state["desc"], state["x"], state["w"], state["y"]))
        return state["y"]
    if kind == "topk":
        _ok(topk.topk_run(state["variant"], state["desc"], state["x"], state["idx"], state["val"]))
        return state["idx"], state["val"]
    for d, A, B, C in state["calls"]:
        _ok(gemm.gemm_run_ex(K4, d, A, B, C))
    return state["outs"]


def work(case):
    """Each operand read once, each result written once; multiply-adds counted as two."""
    kind = case["kind"]
    if kind == "topk":
        b, n, k = case["batch"], case["n"], case["k"]
        return {"bytes": 4 * b * n + 8 * b * k, "flops": 0}
    es = BYTES[case["dtype"]]
    if kind == "conv":
        n, hw, C, F, k, s = (case[x] for x in ("n", "hw", "C", "F", "ksize", "stride"))
        P = (hw + 2 * (k // 2) - k) // s + 1
        return {"bytes": es * (n * hw * hw * C + F * k * k * C + n * P * P * F), "flops": 2 * n * P * P * F * k * k * C}
    if kind == "linear":
        T, I, O = case["tokens"], case["inp"], case["out"]
        # X, W and dY are read by the forward and the backward pass, which a program runs at different times
        return {"bytes": es * 2 * (T * I + O * I + T * O) + 4 * O + es * (T * O + T * I + O * I), "flops": 6 * T * I * O}
    b, M, N, K = case.get("batch", 1), case["M"], case["N"], case["K"]
    return {"bytes": b * (es * (M * K + K * N) + BYTES[OUT[case["dtype"]]] * M * N), "flops": 2 * b * M * N * K}


def tolerance(case):
    if case["kind"] == "topk":
        return "exact"
    return TOLERANCE[OUT[case["dtype"]]]


# About four times what the outputs of the listed cases differ by from the same product in 64 bits (fp32: 8.1e-7 and
# 7.3e-6 at 2048^3; fp16: 2.07e-4 and 4.9e-4; bf16: 1.66e-3 and 3.9e-3, the rounding of the output).
TOLERANCE = {"f32": {"rel": 3.3e-6, "max": 3e-5}, "f16": {"rel": 8.3e-4, "max": 2e-3}, "bf16": {"rel": 6.6e-3, "max": 1.6e-2}}
