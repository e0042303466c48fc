"""Timed work of the library: what a program that serves or converts a model with MX+ operands has it do, through the
Python binding.

Kinds of case (`kind`):
    operands   both operands converted, multiplied and one converted back: the whole path, on small matrices
    decode     a linear layer in the decode stage: few rows of bf16 activations, weights in the 4-bit image of their format
    canonical  the same with the weights left in their canonical bytes (no second copy of them)
    weight_only  bf16 activations as they are x canonical weights of any format (few rows: decode; many: prefill)
    linear     a linear layer in the prefill stage: bf16 activations converted on the fly, weights in their image
    step       the prefill layer with every stage: activations -> canonical + image and weights -> image in one launch,
               product, activations back to bf16; all buffers kept by the caller
    product    the product of two images that are both at hand
    gemm       the product from canonical operands, any pair of formats (builds what the kernels need in its workspace)
    convert    a weight or activation tensor into canonical bytes (rows along K, or K-strided "[K][N]" storage)
    roundtrip  a tensor into canonical bytes and back
Inputs are drawn on the GPU from the case's seed: activations N(0, 1) with outlier channels x 50, weights N(0, 0.02^2)
with 0.1 % of heavy-tailed Student-t(3) entries, as in the synthetic workloads of the package.
"""
import math

import torch

from paper_2510_14557_amd import mxp

BITS = {"MXFP4": 4, "MXFP4P": 4, "MXFP4PP": 4, "MXFP6": 6, "MXFP6P": 6, "MXFP8": 8, "MXFP8P": 8}
FORMATS = tuple(BITS)
DTYPES = {"f32": torch.float32, "bf16": torch.bfloat16}
SIZE = {"f32": 4, "bf16": 2}


def fmt(name):
    return getattr(mxp, name)


def listed():
    return [
        # the smallest call: the tiny fp32 configuration, every entry point of the plain path once (launches and host time)
        {"name": "tiny operands", "kind": "operands", "M": 16, "N": 256, "K": 256, "src": "f32", "out": "f32"},
        # decode, 8 sequences, an attention projection of an 8B-sized model, MXFP4+ weights in their 4-bit image
        {"name": "decode attention", "kind": "decode", "M": 8, "N": 4096, "K": 4096, "w": "MXFP4P", "out": "bf16"},
        # decode, 8 sequences, an MLP layer of a 70B-sized model, weights only in canonical storage
        {"name": "decode 70B canonical", "kind": "canonical", "M": 8, "N": 28672, "K": 8192, "w": "MXFP4P", "out": "bf16"},
        # decode with weight-only quantization, an odd batch, an MLP layer of an 8B-sized model
        {"name": "decode weight-only", "kind": "weight_only", "M": 13, "N": 14336, "K": 4096, "w": "MXFP4P", "out": "bf16"},
        # prefill of 2048 tokens, q / o projection of an 8B-sized model
        {"name": "prefill attention", "kind": "linear", "M": 2048, "N": 4096, "K": 4096, "w": "MXFP4P", "out": "bf16"},
        # prefill of 4096 tokens, gate / up projection, every stage: the step of the benchmark
        {"name": "prefill MLP step", "kind": "step", "M": 4096, "N": 14336, "K": 4096, "w": "MXFP4P", "out": "f32"},
        # the same layer with weight-only quantization
        {"name": "prefill weight-only", "kind": "weight_only", "M": 4096, "N": 14336, "K": 4096, "w": "MXFP4P", "out": "bf16"},
        # the largest product: a 70B-sized layer over 8192 tokens
        {"name": "prefill 70B product", "kind": "product", "M": 8192, "N": 28672, "K": 8192, "w": "MXFP4P", "out": "f32"},
        # ragged sizes and finer activations: MXFP4++ rows on MXFP4+ weights, from canonical bytes
        {"name": "ragged MXFP4++ gemm", "kind": "gemm", "M": 1037, "N": 3001, "K": 4128, "a": "MXFP4PP", "w": "MXFP4P", "out": "f32"},
        # eight-bit operands with extended block maxima, from canonical bytes
        {"name": "MXFP8+ gemm", "kind": "gemm", "M": 2048, "N": 4096, "K": 4096, "a": "MXFP8P", "w": "MXFP8P", "out": "f32"},
        # loading a model: a 70B-sized weight matrix into canonical MXFP4+
        {"name": "convert 70B weights", "kind": "convert", "rows": 28672, "K": 8192, "f": "MXFP4P", "src": "bf16", "strided": False},
        # six-bit storage of an activation-sized tensor and back
        {"name": "roundtrip MXFP6+", "kind": "roundtrip", "rows": 4096, "K": 14336, "f": "MXFP6P", "src": "bf16", "dst": "bf16"},
    ]


def _spread(rng, lo, hi, step=1):
    """A multiple of `step` between lo and hi, even over the logarithm."""
    v = math.exp(rng.uniform(math.log(lo), math.log(hi)))
    return min(max(int(round(v / step)) * step, lo), hi)


def draw(rng):
    kind = rng.choice(("operands", "decode", "canonical", "weight_only", "weight_only", "linear", "step", "product", "gemm", "gemm",
                       "convert", "roundtrip"))
    out = rng.choice(("f32", "bf16"))
    four = rng.choice(("MXFP4", "MXFP4P", "MXFP4P", "MXFP4PP"))
    two = rng.choice(("MXFP4", "MXFP4P", "MXFP4P"))
    if kind == "operands":
        return {"kind": kind, "M": _spread(rng, 1, 256), "N": _spread(rng, 16, 1024), "K": _spread(rng, 32, 1024, 32),
                "src": rng.choice(("f32", "bf16")), "out": out}
    if kind == "decode":
        return {"kind": kind, "M": _spread(rng, 1, 64), "N": _spread(rng, 1000, 28672), "K": _spread(rng, 1024, 14336, 32), "w": four, "out": out}
    if kind == "canonical":
        return {"kind": kind, "M": _spread(rng, 1, 64), "N": _spread(rng, 1000, 28672), "K": _spread(rng, 1024, 14336, 256), "w": two, "out": out}
    if kind == "weight_only":
        few = rng.random() < 0.5
        w = rng.choice(("MXFP4", "MXFP4P", "MXFP4P", "MXFP4PP") if few else FORMATS)
        return {"kind": kind, "M": _spread(rng, 1, 64) if few else _spread(rng, 65, 4096), "N": _spread(rng, 1000, 14336),
                "K": _spread(rng, 1024, 14336 if few else 6144, 32), "w": w, "out": out}
    if kind in ("linear", "step", "product"):
        M, N, K = _spread(rng, 129, 8192), _spread(rng, 1000, 14336), _spread(rng, 1024, 14336, 32)
        return {"kind": kind, "M": M, "N": N, "K": K, "w": two, "out": out}
    if kind == "gemm":
        return {"kind": kind, "M": _spread(rng, 1, 2048), "N": _spread(rng, 1000, 8192), "K": _spread(rng, 1024, 8192, 32),
                "a": rng.choice(FORMATS), "w": rng.choice(FORMATS), "out": out}
    rows, K = _spread(rng, 1, 14336), _spread(rng, 1024, 14336, 32)
    if kind == "convert":
        strided = rng.random() < 0.4
        if strided:
            rows = max(8, rows // 8 * 8)
        return {"kind": kind, "rows": rows, "K": K, "f": four if strided else rng.choice(FORMATS), "src": rng.choice(("f32", "bf16", "bf16")),
                "strided": strided}
    return {"kind": kind, "rows": rows, "K": K, "f": rng.choice(FORMATS), "src": rng.choice(("f32", "bf16", "bf16")),
            "dst": rng.choice(("f32", "bf16"))}


def _activations(rows, K, gen, dtype):
    x = torch.randn((rows, K), generator=gen, device="cuda")
    ch = torch.randint(0, K, (max(2, round(8 * K / 4096)),), generator=gen, device="cuda")
    x[:, ch] *= 50.0
    return x.to(dtype)


def _weights(N, K, gen, dtype=torch.bfloat16):
    w = torch.randn((N, K), generator=gen, device="cuda").mul_(0.02)
    n = max(1, N * K // 1000)
    z = torch.randn((4, n), generator=gen, device="cuda")
    t3 = z[0] / torch.sqrt((z[1] ** 2 + z[2] ** 2 + z[3] ** 2) / 3.0)
    at = (torch.arange(n, device="cuda") * 1000 + torch.randint(0, 1000, (n,), generator=gen, device="cuda")).clamp_(max=N * K - 1)
    w.view(-1)[at] = t3 * 0.2
    return w.to(dtype)


def _inputs(case, seed):
    """(activations or None, weights) of a case, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    if case["kind"] in ("convert", "roundtrip"):
        return None, _weights(case["rows"], case["K"], gen, DTYPES[case["src"]])
    dt = DTYPES[case.get("src", "bf16")]
    W = _weights(case["N"], case["K"], gen, dt)
    return _activations(case["M"], case["K"], gen, dt), W


def prepare(case, seed):
    s = dict(case)
    kind = case["kind"]
    A, W = _inputs(case, seed)
    if kind == "operands":
        s["A"], s["W"] = A, W
    elif kind in ("convert", "roundtrip"):
        s["X"] = W.t().contiguous() if case.get("strided") else W
    else:
        M, N, K, w = case["M"], case["N"], case["K"], fmt(case["w"])
        qw = mxp.quantize(W, w)
        if kind == "decode":
            s["A"] = A
            if case["w"] == "MXFP4":
                s["image"], s["b_kind"] = mxp.prepack_e2m1(qw), mxp.IMAGE_E2M1
            elif case["w"] == "MXFP4P":
                s["image"], s["b_kind"] = mxp.prepack_e2m1r(qw), mxp.IMAGE_E2M1R
            else:
                s["image"], s["b_kind"] = mxp.prepack_e2m1x(qw, w), mxp.IMAGE_E2M1X
        elif kind == "linear" or kind == "product":
            plain = case["w"] == "MXFP4"
            s["image"], s["b_kind"] = (mxp.prepack_e2m1(qw), mxp.IMAGE_E2M1) if plain else (mxp.prepack(qw, w), mxp.IMAGE_E2M3)
            if kind == "linear":
                s["A"] = A
            else:
                s["a_image"] = mxp.quantize_image(A, mxp.MXFP4P)
        elif kind == "step":
            u8 = dict(dtype=torch.uint8, device="cuda")
            s["A"], s["qw"] = A, qw
            s["qa"] = (torch.empty((M, K // 2), **u8), torch.empty((M, K // 32), **u8), torch.empty((M, K // 32), **u8))
            s["a_image"], s["image"] = torch.empty(mxp.image_bytes(M, K), **u8), torch.empty(mxp.image_bytes(N, K), **u8)
            s["D"] = torch.empty((M, N), dtype=DTYPES[case["out"]], device="cuda")
            s["back"] = torch.empty((M, K), dtype=torch.bfloat16, device="cuda")
        elif kind == "gemm":
            s["qa"], s["qw"] = mxp.quantize(A, fmt(case["a"])), qw
        else:                                              # canonical, weight_only
            s["A"], s["qw"] = A, qw
    return s


def _canonical(q, f):
    """The arrays that the format has: the plain forms write no index bytes."""
    return q if f.endswith("P") else q[:2]


def run(s):
    kind = s["kind"]
    if kind == "operands":
        qa, qw = mxp.quantize(s["A"], mxp.MXFP4P), mxp.quantize(s["W"], mxp.MXFP4P)
        return qa, qw, mxp.gemm(qa, mxp.MXFP4P, qw, mxp.MXFP4P, DTYPES[s["out"]]), mxp.dequantize(qa, mxp.MXFP4P, s["A"].dtype)
    if kind == "decode" or kind == "linear":
        return mxp.gemm_bf16a(s["A"], mxp.MXFP4P, s["image"], s["N"], DTYPES[s["out"]], b_kind=s["b_kind"])
    if kind == "canonical":
        return mxp.gemm_decode_bf16a(s["A"], mxp.MXFP4P, s["qw"], fmt(s["w"]), DTYPES[s["out"]])
    if kind == "weight_only":
        return mxp.gemm_w4a16(s["A"], s["qw"], fmt(s["w"]), DTYPES[s["out"]])
    if kind == "step":
        mxp.convert_operands(s["A"], mxp.MXFP4P, s["qa"], s["a_image"], s["qw"], fmt(s["w"]), s["image"])
        mxp.gemm_prepacked(s["M"], s["N"], s["K"], s["a_image"], s["image"], out=s["D"])
        mxp.dequantize(s["qa"], mxp.MXFP4P, out=s["back"])
        return s["qa"], s["D"], s["back"]
    if kind == "product":
        return mxp.gemm_prepacked(s["M"], s["N"], s["K"], s["a_image"], s["image"], DTYPES[s["out"]], b_kind=s["b_kind"])
    if kind == "gemm":
        return mxp.gemm(s["qa"], fmt(s["a"]), s["qw"], fmt(s["w"]), DTYPES[s["out"]])
    f = s["f"]
    q = mxp.quantize_t(s["X"], fmt(f)) if s.get("strided") else mxp.quantize(s["X"], fmt(f))
    if kind == "convert":
        return _canonical(q, f)
    return _canonical(q, f), mxp.dequantize(q, fmt(f), DTYPES[s["dst"]])


# Element grid of a format: significand bits behind the point, smallest exponent, largest magnitude, e_max; and the bits that
# the + forms give the block maximum (its exponent is e_max).
GRID = {"MXFP4": (1, 0, 6.0, 2), "MXFP6": (3, 0, 7.5, 2), "MXFP8": (3, -6, 448.0, 8)}
BM_BITS = {"MXFP4": 3, "MXFP6": 5, "MXFP8": 7}


def _exponent(v):
    """floor(log2 |v|), far down for zero."""
    return torch.where(v == 0, -1000, torch.frexp(v)[1] - 1)


def _scaled(v, e):
    """v * 2^e, from the exponent's bits (exact for results in the normal range)."""
    return v * ((e.long().clamp(-1022, 1023) + 1023) << 52).view(torch.float64)


def _represented(x, f):
    """The values, in 64 bits, that a tensor has in format f: blocks of 32 along the rows with the shared exponent
    floor(log2 max) - e_max, elements to the nearest (ties to even, saturating); in the + forms the first element of
    largest magnitude keeps the block's exponent and more significand bits; in the ++ form the others take a scale of
    their own, up to seven steps finer, that keeps the largest of them below 4."""
    base = f.rstrip("P")
    bits, low, top, e_max = GRID[base]
    v = x.double().view(x.shape[0], -1, 32)
    at = v.abs().max(dim=2, keepdim=True).values
    is_bm = torch.arange(32, device=v.device) == (v.abs() == at).to(torch.uint8).argmax(dim=2, keepdim=True)
    e = _exponent(at)
    shared = e - e_max
    scale = shared
    if f.endswith("PP"):
        rest = _exponent(v.abs().masked_fill(is_bm, 0.0).max(dim=2, keepdim=True).values)
        scale = torch.minimum(torch.maximum(torch.maximum(rest - 1, shared - 7), torch.full_like(shared, -126)), shared)
    u = _scaled(v, -scale)
    step = _exponent(u).clamp(min=low) - bits
    q = _scaled(_scaled(torch.round(_scaled(u, -step)), step).clamp(-top, top), scale)
    if f.endswith("P"):
        n = BM_BITS[base]
        m = torch.round(_scaled(v, n - e)).clamp(-(2.0 ** (n + 1) - 1), 2.0 ** (n + 1) - 1)
        q = torch.where(is_bm, _scaled(m, e - n), q)
    return torch.where(e <= e_max - 127, 0.0, q).view(x.shape)


def exact(case, seed):
    """What run() computes, in 64 bits and without the package; None for bytes, which have no such value."""
    kind = case["kind"]
    if kind == "convert":
        return None
    A, W = _inputs(case, seed)
    none3 = (None, None, None)
    if kind == "roundtrip":
        return _canonical(none3, case["f"]), _represented(W, case["f"])
    a = A.double() if kind == "weight_only" else _represented(A, case.get("a", "MXFP4P"))
    D = a @ _represented(W, case.get("w", "MXFP4P")).t()
    if kind == "operands":
        return none3, none3, D, a
    return (none3, D, a) if kind == "step" else D


def _operand_bytes(rows, K, f):
    """Canonical bytes of an operand: codes, a scale byte per block and, for the + forms, an index byte."""
    return rows * K * BITS[f] / 8 + rows * (K // 32) * (2 if f.endswith("P") else 1)


def work(case):
    kind = case["kind"]
    if kind in ("convert", "roundtrip"):
        n = case["rows"] * case["K"]
        b = n * SIZE[case["src"]] + _operand_bytes(case["rows"], case["K"], case["f"])
        return {"bytes": b + (n * SIZE[case["dst"]] if kind == "roundtrip" else 0), "flops": 0.0}
    M, N, K = case["M"], case["N"], case["K"]
    flops, out = 2.0 * M * N * K, M * N * SIZE[case["out"]]
    if kind == "operands":
        b = (M + N) * K * SIZE[case["src"]] + _operand_bytes(M, K, "MXFP4P") + _operand_bytes(N, K, "MXFP4P") + out + M * K * SIZE[case["src"]]
    elif kind == "gemm":
        b = _operand_bytes(M, K, case["a"]) + _operand_bytes(N, K, case["w"]) + out
    elif kind == "product":
        b = M * K * 25 / 32 + N * K * (17 if case["w"] == "MXFP4" else 25) / 32 + out
    elif kind == "linear":
        b = M * K * 2 + N * K * (17 if case["w"] == "MXFP4" else 25) / 32 + out
    elif kind == "step":
        b = M * K * 4 + _operand_bytes(M, K, "MXFP4P") + _operand_bytes(N, K, case["w"]) + out
    else:
        b = M * K * 2 + _operand_bytes(N, K, case["w"]) + out
    return {"bytes": b, "flops": flops}


def tolerance(case):
    """Bytes of a conversion are fixed by the format; so is every de-converted value.  A product is exact up to its fp32 sum
    (against sums in 64 bits: up to 1.8e-7, largest 1.5e-6); with bf16 output a last bit may round the other way (4.1e-5; one
    unit is at most 2^-7 of the value); two MXFP4++ operands meet on the FP8 matrix instruction, which drops low bits of the
    smaller products of a group (1.2e-5, largest 1.7e-4).  About four times that is allowed."""
    if case["kind"] in ("convert", "roundtrip"):
        return "exact"
    if case["out"] == "bf16":
        return {"rel": 2e-4, "max": 8e-3}
    if case.get("a") == "MXFP4PP" and case.get("w") == "MXFP4PP":
        return {"rel": 5e-5, "max": 7e-4}
    return {"rel": 8e-7, "max": 8e-6}
