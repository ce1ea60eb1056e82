"""The workloads by which the speed of the quantized linears is judged.

A case is one pass over what a user of this library runs per layer: the four linears of a Visual-Mamba
block (in_proj, x_proj, dt_proj, out_proj, each on its own resident activations, as in bench.py), or one
linear of free widths.  Weights are folded and quantized beforehand and stay in memory, like the codes'
and the outputs' buffers; a pass is the activation quantizer and the linear, in the launch form that
include/ptq4vm.h recommends for the shape:

  w8a8     PTS quantizer + W8A8 linear; one fused launch for narrow outputs (N <= 128, >= 4096 rows)
           and short reductions (K <= 128, >= 16384 rows)
  w4a4     one fused launch where the 4-bit form has one, else the E2M3 container where K fills whole
           blocks of 128 codes, else packed nibbles
  offset   W8A8 with a per-token zero offset; one fused launch where that form has one
  dynamic  per-token dynamic quantizer + W8A8 linear
  f16      the unquantized linear

Row counts are images times tokens: 197 tokens are 224 x 224 pixels in patches of 16 plus the class token,
785 the same picture at stride 8.
"""
from __future__ import annotations

import math

import torch

import paper_2412_20386_amd as ptq
from paper_2412_20386_amd import synth

DEVICE = "cuda:0"
BLOCKS = {"ti": synth.CONFIGS[1].linears, "s": synth.CONFIGS[2].linears, "b": synth.CONFIGS[3].linears}
MAX_ROWS = 50432  # the largest batch of the benchmark: 256 images of 197 tokens


def _block(name, scheme, size, B, L):
    return dict(name=name, kind="block", scheme=scheme, size=size, B=B, L=L)


def _linear(name, scheme, K, N, B, L):
    return dict(name=name, kind="linear", scheme=scheme, K=K, N=N, B=B, L=L)


def listed():
    return [
        # the smallest call: one projection of the smallest model for one image
        _linear("ti_out_proj_1_image", "w8a8", 384, 192, 1, 197),
        # one image through a block of the largest model: serving latency
        _block("b_block_1_image", "w8a8", "b", 1, 197),
        # the benchmark's stacks, one block each: small, medium, long sequence, largest
        _block("ti_block_64_images", "w8a8", "ti", 64, 197),
        _block("s_block_128_images", "w8a8", "s", 128, 197),
        _block("s_block_64_long_images", "w8a8", "s", 64, 785),
        _block("b_block_256_images", "w8a8", "b", 256, 197),
        # 4-bit codes: an ordinary serving batch and the benchmark's largest
        _block("s_block_16_images_w4a4", "w4a4", "s", 16, 197),
        _block("b_block_256_images_w4a4", "w4a4", "b", 256, 197),
        # steps computed online, an ordinary batch
        _block("s_block_32_images_dynamic", "dynamic", "s", 32, 197),
        # asymmetric activations: a zero offset per token
        _block("b_block_64_images_offset", "offset", "b", 64, 197),
        # the unquantized model
        _block("s_block_128_images_f16", "f16", "s", 128, 197),
        # widths that are no multiple of anything the kernels tile by (pruned or odd-sized layers)
        _linear("ragged_linear", "w8a8", 1000, 500, 16, 199),
    ]


def _log_uniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    scheme = rng.choice(["w8a8"] * 5 + ["w4a4"] * 2 + ["dynamic", "offset", "f16"])
    # the slower schemes stop at half the rows, so that no drawn case costs more than the largest listed one
    rows = MAX_ROWS if scheme in ("w8a8", "w4a4") else MAX_ROWS // 2
    L = _log_uniform(rng, 49, 1025)
    if rng.random() < 0.75:
        B = _log_uniform(rng, 1, max(1, rows // L))
        return dict(kind="block", scheme=scheme, size=rng.choice(["ti", "s", "b"]), B=B, L=L)
    B = _log_uniform(rng, 1, max(1, rows // 2 // L))
    K, N = _log_uniform(rng, 24, 2048), _log_uniform(rng, 16, 3072)
    if rng.random() < 0.5:  # half of the layers keep widths that are multiples of 64
        K, N = max(64, K // 64 * 64), max(64, N // 64 * 64)
    if scheme == "w4a4":
        K += K % 2  # packed nibbles need an even reduction length
    return dict(kind="linear", scheme=scheme, K=K, N=N, B=B, L=L)


def _shapes(case):
    if case["kind"] == "linear":
        return [(case["K"], case["N"])]
    return [(K, N) for _, K, N in BLOCKS[case["size"]]]


def _form(scheme, M, K, N):
    """The launch form of one linear: "fused" (one launch), "two" (quantizer, then linear), "e2m3", "f16" or "dynamic"."""
    if scheme in ("f16", "dynamic"):
        return scheme
    if scheme == "w8a8":
        return "fused" if (N <= 128 and M >= 4096) or (K <= 128 and M >= 16384) else "two"
    # the one-launch 4-bit and offset forms exist where the weight fits on chip; other shapes take two launches
    if N <= 128 and K % 64 == 0 and M >= 4096 and ((N <= 80 and K <= 1536) or N * K <= 128 * 768):
        return "fused"
    if M >= 16384 and ((K <= 64 and N <= 1536) or (K <= 128 and N <= 768)):
        return "fused"
    return "e2m3" if scheme == "w4a4" and K % 128 == 0 and K >= 256 else "two"


def prepare(case, seed):
    B, L, scheme = case["B"], case["L"], case["scheme"]
    M = B * L
    steps = []
    for i, (K, N) in enumerate(_shapes(case)):
        c = synth.random_problem(seed * 16 + i, B, L, K, N, device=DEVICE)
        form = _form(scheme, M, K, N)
        d = dict(form=form, scheme=scheme, B=B, L=L, M=M, K=K, x=c.x, bias=c.bias, s_tok=c.s_tok,
                 y=torch.empty((M, N), dtype=torch.float16, device=DEVICE))
        if scheme == "f16":
            d["w"] = c.w
        elif scheme == "w4a4":
            d["s_tok"] = c.s_tok * (127.0 / 7.0)
            if form == "e2m3":
                d["wq"], d["s_w"], d["inv_m"] = ptq.fold_smoothing_w4_e2m3(c.w, c.m)
                d["xq"] = torch.empty((ptq.e2m3_blocks(K), M, 96), dtype=torch.uint8, device=DEVICE)
            else:
                d["wq"], d["s_w"], d["inv_m"] = ptq.fold_smoothing_w4(c.w, c.m)
                d["xq"] = torch.empty((M, K // 2), dtype=torch.uint8, device=DEVICE)
        else:
            d["wq"], d["s_w"], d["inv_m"] = ptq.fold_smoothing(c.w, c.m)
            d["xq"] = torch.empty((M, K), dtype=torch.int8, device=DEVICE)
            if scheme == "dynamic":
                d["s_row"] = torch.empty(M, dtype=torch.float32, device=DEVICE)
            if scheme == "offset":
                d["x"] = (c.x.view(B, L, K) + synth.token_shift(L, seed, DEVICE).view(1, L, 1)).view(M, K)
                d["s_tok"], d["z_tok"] = synth.calibrate_offset(d["x"], c.m, L)
                d["rowsum"] = ptq.weight_rowsum(d["wq"])
        steps.append(d)
    return steps


def _run_linear(d):
    B, L, form = d["B"], d["L"], d["form"]
    if form == "f16":
        return [ptq.f16_linear(d["x"], d["w"], d["bias"], y=d["y"])]
    if form == "dynamic":
        xq, s_row = ptq.quantize_dynamic(d["x"], d["inv_m"], xq=d["xq"], s_row=d["s_row"])
        return [xq, s_row, ptq.w8a8_linear(xq, d["wq"], s_row, d["s_w"], d["bias"], 1, d["M"], y=d["y"])]
    if d["scheme"] == "w8a8":
        if form == "fused":
            return [ptq.w8a8_linear_fused(d["x"], d["inv_m"], d["s_tok"], d["wq"], d["s_w"], d["bias"], B, L, y=d["y"])]
        xq = ptq.quantize_pts(d["x"], d["inv_m"], d["s_tok"], B, L, xq=d["xq"])
        return [xq, ptq.w8a8_linear(xq, d["wq"], d["s_tok"], d["s_w"], d["bias"], B, L, y=d["y"])]
    if d["scheme"] == "offset":
        if form == "fused":
            return [ptq.w8a8_linear_offset_fused(d["x"], d["inv_m"], d["s_tok"], d["z_tok"], d["wq"], d["rowsum"],
                                                 d["s_w"], d["bias"], B, L, y=d["y"])]
        xq = ptq.quantize_pts_offset(d["x"], d["inv_m"], d["s_tok"], d["z_tok"], B, L, xq=d["xq"])
        return [xq, ptq.w8a8_linear_offset(xq, d["wq"], d["s_tok"], d["z_tok"], d["rowsum"], d["s_w"], d["bias"], B, L,
                                           y=d["y"])]
    if form == "fused":
        return [ptq.w4a4_linear_fused(d["x"], d["inv_m"], d["s_tok"], d["wq"], d["s_w"], d["bias"], B, L, y=d["y"])]
    if form == "e2m3":
        xq = ptq.quantize_pts_a4_e2m3(d["x"], d["inv_m"], d["s_tok"], B, L, xq6=d["xq"])
        return [xq, ptq.w4a4_linear_e2m3(xq, d["wq"], d["s_tok"], d["s_w"], d["bias"], B, L, d["K"], y=d["y"])]
    xq = ptq.quantize_pts_a4(d["x"], d["inv_m"], d["s_tok"], B, L, xq4=d["xq"])
    return [xq, ptq.w4a4_linear(xq, d["wq"], d["s_tok"], d["s_w"], d["bias"], B, L, y=d["y"])]


def run(state):
    """The codes (where the form writes them) and the outputs of every linear."""
    return [_run_linear(d) for d in state]


def work(case):
    """Activations, weights, biases and scale vectors in, codes (where they are an output) and results out, once each."""
    M, L = case["B"] * case["L"], case["L"]
    nbytes = flops = 0
    for K, N in _shapes(case):
        form = _form(case["scheme"], M, K, N)
        code = {"e2m3": 0.75, "f16": 2.0}.get(form, 0.5 if case["scheme"] == "w4a4" else 1.0)  # bytes per weight / code
        nbytes += 2 * M * K + code * N * K + 2 * N + 2 * M * N
        if form != "f16":
            nbytes += 4 * K + 4 * N + (4 * M if form == "dynamic" else 4 * L)
            if form != "fused":
                nbytes += code * M * K
        flops += 2 * M * K * N
    return {"bytes": int(nbytes), "flops": flops}


def tolerance(case):
    """Codes, accumulators and dynamic steps have one correct value; outputs are rounded to fp16 once.

    Measured against the same product in 64 bits, not rounded: relative error 2.0e-4 to 2.2e-4 (the rounding to
    fp16 alone), largest difference 4.9e-4 of the value (half an fp16 ulp)."""
    return {"rel": 1e-3, "max": 2e-3}
