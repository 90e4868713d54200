"""What this library is timed on: the passes its users make, over the range of sizes they make them at.

A case is one pass through the public entry points of paper_2511_04214_amd.  Four kinds:

  linear    one rotated, quantized linear layer: the online step on the activations
            (rotate_quantize_fused, or swiglu_rotate_quantize_fused in front of a down-projection), then
            the product with weights that were quantized once (mxfp4_gemm); or both in the one-launch call
            for a few rows (rotate_quantize_gemm_fused)
  quantize  the online step alone: long activations, or weights on their way to a quantized model
  matrix    the online step with caller-supplied orthogonal 32 x 32 blocks
  analysis  the block statistics before and after a rotation and their summary

A user's program keeps the quantized weights, the sign vector and the rotation blocks, and, because an
operand's size is fixed by the layer, the operand buffers that the online step fills; the product's result
is a new tensor each time.
"""
import math

import torch

import paper_2511_04214_amd as brq

_DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}
_THRESHOLDS = (1.5, 3.0)
_EDGES = (1.0, 2.0, 4.0, 8.0, 16.0, 32.0, 64.0)
_OUTLIER = 60.0


def _linear(name, M, N, K, B=32, dtype="bf16", out="bf16", layout="tiled", step="two", signs=False):
    c = dict(kind="linear", M=M, N=N, K=K, B=B, dtype=dtype, out=out, layout=layout, step=step, signs=signs)
    return dict(c, name=name) if name else c


def _quantize(name, M, K, B=32, dtype="bf16", layout="tiled", signs=False):
    c = dict(kind="quantize", M=M, K=K, B=B, dtype=dtype, layout=layout, signs=signs)
    return dict(c, name=name) if name else c


def _matrix(name, M, K, dtype="bf16", layout="tiled"):
    c = dict(kind="matrix", M=M, K=K, dtype=dtype, layout=layout)
    return dict(c, name=name) if name else c


def _analysis(name, M, K, B=32):
    c = dict(kind="analysis", M=M, K=K, B=B)
    return dict(c, name=name) if name else c


def listed():
    return [
        # the smallest layer: one workgroup's worth of work, every argument at its default (fp32, row-major)
        _linear("tiny_default", 16, 256, 256, dtype="f32", out="f32", layout="rowmajor"),
        # generation of one sequence: one row against 28672 x 8192 weights, in the one-launch call
        _linear("decode_1", 1, 28672, 8192, step="one"),
        # generation of a ragged batch of sequences, the same weights
        _linear("decode_batch_100", 100, 28672, 8192),
        # a short prompt, or a chunk of one, the same weights
        _linear("chunk_300", 300, 28672, 8192),
        # a 1B model's up-projection over 2048 tokens
        _linear("prompt_up_2048", 2048, 8192, 2048),
        # a down-projection over 4096 tokens with the global rotation (B = K)
        _linear("prompt_down_global", 4096, 2048, 8192, B=8192),
        # an 8B model's MLP product over 8192 tokens: the largest
        _linear("prompt_mlp_8192", 8192, 14336, 4096),
        # a down-projection with its gated activation fused in, ragged rows, K not a multiple of 512
        _linear("swiglu_down_1000", 1000, 4096, 11008, step="swiglu"),
        # the same weights with the library's defaults: fp32 in, row-major operands, fp32 out
        _linear("default_k11008", 2000, 4096, 11008, dtype="f32", out="f32", layout="rowmajor"),
        # the online step alone over a long batch
        _quantize("rotate_quant_16384", 16384, 8192),
        # ... with learned rotation blocks, one per group
        _matrix("matrix_quant_16384", 16384, 8192),
        # the paper's comparison of block scales and losses before and after the block rotation
        _analysis("analysis_16384", 16384, 8192),
    ]


def _log(rng, lo, hi):
    return math.exp(rng.uniform(math.log(lo), math.log(hi)))


def _block(rng, K):
    """Mostly the method's 32; the wider blocks of its sweep; the global rotation where K allows it."""
    some = [32, 32, 32] + [b for b in (64, 128) if K % b == 0]
    if K & (K - 1) == 0 and 256 <= K <= 16384:
        some.append(K)
    return rng.choice(some)


def _k(rng, hi, unit=None):
    unit = unit or rng.choice([32, 128, 128, 512, 512, 512])
    if rng.random() < 0.2:
        return 2 ** rng.randrange(9, int(math.log2(hi)) + 1)
    return max(unit, int(_log(rng, 256, hi)) // unit * unit)


def draw(rng):
    kind = rng.choice(["linear"] * 7 + ["quantize", "matrix", "analysis"])
    dtype = rng.choice(["bf16"] * 4 + ["f32"])
    layout = rng.choice(["tiled", "tiled", "rowmajor"])
    signs = rng.random() < 0.2
    if kind == "linear":
        out = rng.choice(["bf16"] * 3 + ["f32"])
        step = rng.choice(["two"] * 6 + ["swiglu"] * 2 + ["one"])
        while True:
            N = int(_log(rng, 256, 28672))
            N = N if rng.random() < 0.1 else N // 8 * 8
            if step == "one":     # its contract: M <= 16, K % 512 == 0, K <= 16384, B = 32; it is meant for a few rows
                M, K, B = rng.randrange(1, 4), _k(rng, 16384, 512), 32
            else:
                M, K = int(_log(rng, 1, 8192)), _k(rng, 14336)
                B = _block(rng, K)
            big = 8192 * 14336 * 4096 if layout == "tiled" and N % 8 == 0 else 2000 * 4096 * 11008
            if M * N * K <= big and M * K <= 8192 * 8192 and N * K <= 28672 * 8192:
                return _linear(None, M, N, K, B=B, dtype=dtype, out=out, layout=layout, step=step, signs=signs)
    if kind == "quantize":
        K = _k(rng, 16384)
        M = int(_log(rng, 16, 16384 * 8192 / K))
        return _quantize(None, min(M, 28672), K, B=_block(rng, K), dtype="bf16" if M * K > 2 ** 26 else dtype, layout=layout, signs=signs)
    if kind == "matrix":
        K = _k(rng, 14336, 128)
        M = int(_log(rng, 16, 16384 * 8192 / K))
        return _matrix(None, min(M, 28672), K, dtype="bf16" if M * K > 2 ** 24 else dtype, layout=layout)
    K = _k(rng, 14336)
    M = int(_log(rng, 16, 16384 * 8192 / K))
    return _analysis(None, min(M, 28672), K, B=_block(rng, K))


def _activations(g, M, K, dtype):
    """Heavy-tailed rows (Student t with 4 degrees of freedom) with 1 % of the channels twenty times as large."""
    u = torch.rand((2, M, K), generator=g, device="cuda").clamp_(min=1e-30)
    x = u[0].log_().add_(u[1].log_()).mul_(-0.5).rsqrt_()       # 1 / sqrt(chi-squared_4 / 4)
    del u
    x.mul_(torch.randn((M, K), generator=g, device="cuda"))
    cols = torch.randperm(K, generator=g, device="cuda")[: max(1, K // 100)]
    x[:, cols] *= 20.0
    return x.to(_DTYPES[dtype])


def _operand_buffers(M, K, layout):
    cb, sb = brq.operand_bytes(M, K, layout)
    shapes = ((M, K // 2), (M, K // 32)) if layout == "rowmajor" else ((cb,), (sb,))
    return [torch.zeros(s, dtype=torch.uint8, device="cuda") for s in shapes]     # (row padding is never written)


def prepare(case, seed):
    g = torch.Generator(device="cuda").manual_seed(seed)
    M, K = case["M"], case["K"]
    s = dict(case=case)
    if case.get("step") == "swiglu":      # gate and up are the two halves of one projection's output
        h = torch.randn((M, 2 * K), generator=g, device="cuda")
        h[:, K:].mul_(_activations(g, M, K, "f32"))
        h = h.to(_DTYPES[case["dtype"]])
        s["gate"], s["up"] = h[:, :K], h[:, K:]
    else:
        s["x"] = _activations(g, M, K, case.get("dtype", "bf16"))
    signs = None
    if case.get("signs"):
        signs = (torch.randint(0, 2, (K,), generator=g, device="cuda") * 2 - 1).to(torch.int8)
    s["signs"] = signs
    if case["kind"] != "analysis":
        s["codes"], s["scales"] = _operand_buffers(M, K, case["layout"])
    if case["kind"] == "linear":
        w = torch.randn((case["N"], K), generator=g, device="cuda").mul_(0.02).to(torch.bfloat16)
        s["wq"], s["ws"] = brq.rotate_quantize_fused(w, case["B"], layout=case["layout"], signs=signs)
    if case["kind"] == "matrix":
        s["R"] = torch.linalg.qr(torch.randn((K // 32, 32, 32), generator=g, device="cuda"))[0].contiguous()
    return s


def run(s):
    c = s["case"]
    kind, layout = c["kind"], c.get("layout")
    if kind == "analysis":
        amax0, above0, loss0 = brq.block_stats(s["x"], 1, thresholds=_THRESHOLDS)
        amax, above, loss = brq.block_stats(s["x"], c["B"], thresholds=_THRESHOLDS)
        hist, counts, sums = brq.block_stats_summary(amax, loss, amax_ref=amax0, outlier_threshold=_OUTLIER, edges=_EDGES)
        return [amax0, above0, loss0, amax, above, loss, hist, counts, sums]
    if kind == "matrix":
        return list(brq.matrix_rotate_quantize_fused(s["x"], s["R"], codes=s["codes"], scales=s["scales"], layout=layout))
    if kind == "quantize":
        return list(brq.rotate_quantize_fused(s["x"], c["B"], codes=s["codes"], scales=s["scales"], layout=layout, signs=s["signs"]))
    out = _DTYPES[c["out"]]
    if c["step"] == "one":
        return [brq.rotate_quantize_gemm_fused(s["x"], c["B"], s["wq"], s["ws"], c["N"], out_dtype=out, w_layout=layout,
                                               signs=s["signs"])]
    if c["step"] == "swiglu":
        codes, scales = brq.swiglu_rotate_quantize_fused(s["gate"], s["up"], c["B"], h_dtype=torch.bfloat16, codes=s["codes"],
                                                         scales=s["scales"], layout=layout, signs=s["signs"])
    else:
        codes, scales = brq.rotate_quantize_fused(s["x"], c["B"], codes=s["codes"], scales=s["scales"], layout=layout,
                                                  signs=s["signs"])
    y = brq.mxfp4_gemm(codes, scales, s["wq"], s["ws"], out_dtype=out, a_layout=layout, w_layout=layout, M=c["M"], N=c["N"],
                       K=c["K"])
    return [codes, scales, y]


def work(case):
    """Inputs once, outputs once; the operand between the two halves of a layer stays on the chip in the ideal case.
    Operations: the product's (the rotation itself is a few additions per element)."""
    M, K = case["M"], case["K"]
    es = 2 if case.get("dtype", "bf16") == "bf16" else 4
    q = 0.5 + 1 / 32                                # bytes per quantized element
    if case["kind"] == "analysis":                  # the activations once, scale and loss per block for each of two
        return {"bytes": M * K * (2 + 2 * 8 / 32), "flops": 0}
    if case["kind"] == "quantize":
        return {"bytes": M * K * (es + q), "flops": 0}
    if case["kind"] == "matrix":
        return {"bytes": M * K * (es + q) + K * 32 * 4, "flops": 2 * M * K * 32}
    N, oes = case["N"], 2 if case["out"] == "bf16" else 4
    x = M * K * es * (2 if case["step"] == "swiglu" else 1)
    return {"bytes": x + N * K * q + M * N * oes, "flops": 2 * M * N * K}


def tolerance(case):
    """Codes, scales and counts are defined bit for bit, except where the interface states an error bound instead
    of an operation sequence (rotation blocks on the matrix cores, the gated activation): there values next to a
    rounding boundary may move.  Measured against 64-bit arithmetic: 2.4e-7 of the code bytes for the former,
    9e-7 for the latter, whose layer's result then moves by 1.4e-4 (largest element 0.0123).  The product is a sum
    in 32 bits in whatever order (on these operands, whose scales span a few binades, it came out exact), the
    bf16 result one rounding of it: a sum that moves across a rounding boundary moves the result by one unit."""
    if case["kind"] == "quantize":
        return "exact"
    if case["kind"] == "matrix":
        return {"rel": 0.0, "max": 0.0, "differ": 2e-6}
    if case["kind"] == "analysis":                  # the loss of a block is a sum of 32 squares in 32 bits (4.6e-8, 1.5e-7)
        return {"rel": 2e-7, "max": 6e-7, "differ": 0.0}
    if case["step"] == "swiglu":
        return {"rel": 6e-4, "max": 5e-2, "differ": 4e-6}
    if case["out"] == "f32":
        return {"rel": 1e-6, "max": 1e-5, "differ": 0.0}
    return {"rel": 1e-4, "max": 8e-3, "differ": 0.0}
