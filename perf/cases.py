"""Work that users have this library do, as a list of timed cases.

Three kinds, each one pass through the entry points of `paper_2502_05003_amd.binding`:

  infer        forward of a layer whose weights were quantized once: quantize the tokens' activations
               (no trust mask), multiply the packed codes.  Decode steps and prefill.
  weight_only  forward with 16-bit activations against 4-bit weights: transform the activations, multiply.
  train        one layer's training step: quantize activations and weights with their masks, forward
               product, both gradient products, both masked inverse transforms.

A case: M tokens, N output channels, K input channels, Hadamard block `block`, `grid` ("int": the
Eq. 1 grid of `bits` bits; "fp4": E2M1) and the dtype of activations and weights.
"""
from __future__ import annotations

import math

import torch

from paper_2502_05003_amd import binding as q

DEV = "cuda:0"

# hidden and MLP widths of this repository's layer configurations and kernels
WIDTHS = (512, 640, 768, 1024, 1280, 1664, 1792, 2048, 2816, 3584, 4096, 4608, 5632, 11008)
MAX_TOKENS = 16384


def _case(kind, M, N, K, block, bits=4, grid="int", dtype="bf16", name=None):
    case = dict(kind=kind, M=M, N=N, K=K, block=block, bits=bits, grid=grid, dtype=dtype)
    return case if name is None else dict(name=name, **case)


def listed():
    return [
        # decoding, one sequence: the smallest call, all latency and launches (1.6B model, MLP up)
        _case("infer", 1, 5632, 2048, 2048, name="decode_one"),
        # decoding, a batch of sequences (1.6B model, MLP down)
        _case("infer", 24, 2048, 5632, 512, name="decode_batch"),
        # one ragged prompt through a 2-bit layer of the 100M model, block 128
        _case("infer", 333, 4096, 1024, 128, bits=2, name="prefill_ragged_2bit"),
        # 8 x 1024 tokens through the 100M model's MLP, full-width transform
        _case("infer", 8192, 4096, 1024, 1024, name="prefill_100m"),
        # one full context through the 7B model's MLP
        _case("infer", 4096, 11008, 4096, 4096, name="prefill_7b"),
        # 16-bit activations against 4-bit weights, a short prompt
        _case("weight_only", 512, 5632, 2048, 2048, name="prefill_weight_only"),
        # the tests' tiny layer, fp32 activations and weights
        _case("train", 256, 512, 512, 512, dtype="f32", name="train_tiny_f32"),
        # the smallest model of the family (hidden 640, MLP 1792: ragged tiles), a micro-batch
        _case("train", 2048, 1792, 640, 128, name="train_small"),
        # a width that is in no configuration here (20 x 128)
        _case("train", 4096, 6912, 2560, 512, name="train_other_width"),
        # the FP4 grid, one sequence of 4096 tokens
        _case("train", 4096, 5632, 2048, 2048, grid="fp4", name="train_fp4"),
        # the 1.6B model's MLP at the benchmark's batch: up- and down-projection
        _case("train", 16384, 2048, 5632, 512, name="train_down_1p6b"),
        _case("train", 16384, 5632, 2048, 2048, name="train_up_1p6b"),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(("infer", "infer", "infer", "train", "train", "weight_only"))
    grid = "fp4" if kind != "weight_only" and rng.random() < 0.2 else "int"
    bits = 4 if grid == "fp4" else rng.choice((4, 4, 4, 3, 2, 1))
    dtype = "f32" if kind == "train" and grid == "int" and rng.random() < 0.2 else "bf16"

    def width(multiple):   # a width of the model family, or any other
        if rng.random() < 0.6:
            return rng.choice(WIDTHS)
        return multiple * max(1, round(_log_uniform(rng, 256, 11008) / multiple))

    K = width(128 if grid == "fp4" else rng.choice((64, 128, 256)))
    widest = K & -K
    block = min(widest, 4096) if rng.random() < 0.8 else min(widest, rng.choice((1, 16, 128)))
    if kind == "infer":       # any number of tokens and channels
        M, N = _log_uniform(rng, 1, MAX_TOKENS), width(rng.choice((1, 8, 64)))
    else:                     # the 16-bit products take multiples of 64
        M, N = 64 * _log_uniform(rng, 2, MAX_TOKENS // 64), width(64)
    # no more than the largest listed case, in operations
    per_token = (6.0 if kind == "train" else 2.0) * N * K
    while M > 64 and M * per_token > 6.0 * 16384 * 5632 * 2048:
        M = max(64, M // 128 * 64)
    return _case(kind, M, N, K, block, bits, grid, dtype)


def _random(seed):
    gen = torch.Generator(device=DEV)
    gen.manual_seed(seed)

    def normal(rows, cols, std, dtype, outliers=0.0, gain=1.0):
        t = torch.randn(rows, cols, generator=gen, device=DEV, dtype=torch.float32).mul_(std)
        count = round(outliers * cols)
        if count:   # whole outlier channels, as activations have
            t[:, torch.randperm(cols, generator=gen, device=DEV)[:count]] *= gain
        return t.to(dtype)

    return normal


def _empty(rows, cols, dtype):
    return torch.empty(rows, cols, dtype=dtype, device=DEV)


def _quantized(rows, cols, code_bits, mask):
    """Buffers for one quantized operand."""
    return dict(codes=_empty(rows, cols * code_bits // 8, torch.uint8),
                scales=torch.empty(rows, dtype=torch.float32, device=DEV),
                mask=_empty(rows, cols // 8, torch.uint8) if mask else None)


def _scratch(nbytes):
    return torch.empty(nbytes, dtype=torch.uint8, device=DEV) if nbytes > 0 else None


def prepare(case, seed):
    kind, M, N, K, bits = case["kind"], case["M"], case["N"], case["K"], case["bits"]
    dtype = torch.float32 if case["dtype"] == "f32" else torch.bfloat16
    fp4 = case["grid"] == "fp4"
    normal = _random(seed)
    state = dict(case)
    state["x"] = normal(M, K, 1.0, dtype, outliers=0.005, gain=50.0)
    w = normal(N, K, 0.02, dtype)
    cb = q.quest_container_bits(bits)
    q.quest_init()
    if kind == "train":
        state.update(w=w, dy=normal(M, N, math.sqrt(1e-3), torch.bfloat16))
        state.update(xq=_quantized(M, K, cb, True), wq=_quantized(N, K, cb, True))
        state.update(gx=_empty(M, K, torch.bfloat16), gw=_empty(N, K, torch.bfloat16),
                     dx=_empty(M, K, torch.bfloat16), dw=_empty(N, K, torch.bfloat16))
        query = q.quest_grad_gemm_fp4_workspace_bytes if fp4 else q.quest_grad_gemm_workspace_bytes
        state["scratch"] = _scratch(max(query(which, M, N, K) for which in (0, 1)))
    else:
        wq = _quantized(N, K, cb, False)
        if fp4:
            q.quest_hadamard_quantize_fp4(w, case["block"], codes=wq["codes"], scales=wq["scales"])
        else:
            q.quest_hadamard_quantize(w, case["block"], bits, codes=wq["codes"], scales=wq["scales"])
        state["wq"] = wq
        if kind == "infer":
            state["xq"] = _quantized(M, K, cb, False)
        else:
            state["xh"] = _empty(M, K, torch.bfloat16)
            state["scratch"] = _scratch(q.quest_weight_only_gemm_workspace_bytes(M, N, K))
    if kind != "weight_only":
        state["product_scratch"] = None if fp4 else _scratch(q.quest_lowbit_gemm_workspace_bytes(M, N, K, bits))
    state["y"] = _empty(M, N, torch.bfloat16)
    return state


def run(s):
    kind, K, block, bits, fp4 = s["kind"], s["K"], s["block"], s["bits"], s["grid"] == "fp4"
    if kind == "weight_only":
        q.quest_trust_backward(s["x"], None, block, out=s["xh"])   # x_h = HT(x)
        q.quest_weight_only_gemm(s["xh"], s["wq"]["codes"], s["wq"]["scales"], bits, y=s["y"],
                                 workspace=s["scratch"])
        return s["y"]

    xq, wq = s["xq"], s["wq"]
    if kind == "infer":
        if fp4:
            q.quest_hadamard_quantize_fp4(s["x"], block, codes=xq["codes"], scales=xq["scales"])
        else:
            q.quest_hadamard_quantize(s["x"], block, bits, codes=xq["codes"], scales=xq["scales"])
    else:
        outputs = dict(x_codes=xq["codes"], x_scales=xq["scales"], x_mask=xq["mask"],
                       w_codes=wq["codes"], w_scales=wq["scales"], w_mask=wq["mask"])
        if fp4:
            q.quest_hadamard_quantize_fp4_pair(s["x"], s["w"], block, **outputs)
        else:
            q.quest_hadamard_quantize_pair(s["x"], s["w"], block, bits, **outputs)
    if fp4:
        q.quest_lowbit_gemm_fp4(xq["codes"], xq["scales"], wq["codes"], wq["scales"], K, y=s["y"])
    else:
        q.quest_lowbit_gemm(xq["codes"], xq["scales"], wq["codes"], wq["scales"], K, bits, y=s["y"],
                            workspace=s["product_scratch"])
    if kind == "infer":
        return s["y"]

    M, N, scratch = s["M"], s["N"], s["scratch"]
    if fp4:
        q.quest_grad_gemm_fp4(0, s["dy"], wq["codes"], wq["scales"], M, N, K, out=s["gx"], workspace=scratch)
        q.quest_grad_gemm_fp4(1, s["dy"], xq["codes"], xq["scales"], M, N, K, out=s["gw"], workspace=scratch)
    else:
        q.quest_grad_gemm(0, s["dy"], wq["codes"], wq["scales"], bits, M, N, K, out=s["gx"], workspace=scratch)
        q.quest_grad_gemm(1, s["dy"], xq["codes"], xq["scales"], bits, M, N, K, out=s["gw"], workspace=scratch)
    q.quest_trust_backward_pair(s["gx"], xq["mask"], s["gw"], wq["mask"], block, out_x=s["dx"], out_w=s["dw"])
    return dict(y=s["y"], dx=s["dx"], dw=s["dw"])


def work(case):
    M, N, K = case["M"], case["N"], case["K"]
    elem = 4 if case["dtype"] == "f32" else 2
    if case["kind"] == "train":   # x, w, dy in; y, dx, dw out
        return dict(bytes=(M + N) * K * (elem + 2) + 4 * M * N, flops=6 * M * N * K)
    code_bits = q.quest_container_bits(case["bits"])
    return dict(bytes=elem * M * K + N * K * code_bits // 8 + 4 * N + 2 * M * N, flops=2 * M * N * K)


def tolerance(case):
    # Against the same path in float64 (13 shapes of all kinds): rel 0.0017 for y (one bf16 rounding)
    # and 0.0029 for the gradients (two); largest single difference 0.01 to 0.10 of the rms, where an
    # activation or weight within 1e-6 of a cell boundary took the neighbouring code.
    return {"rel": 1e-2, "max": 0.25}
