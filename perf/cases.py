"""Timed cases of the library: the calls a program that runs RFQ linear layers
makes, over the range of sizes it makes them at.

A case is a dict of plain values.  "path" names the calls of one pass:

  quantize   activations to primary and residual MXFP4 codes (rfq_quantize_act)
  linear     one quantized linear layer on weights quantized beforehand:
             rfq_quantize_act, then rfq_gemm (with "split", K may be split)
  stream     the same layer in one call, rfq_gemm_stream
  qat        a layer whose fp32 master weight is quantized on every forward:
             rfq_quantize_weight, rfq_quantize_act, rfq_gemm
  phi        a layer with a fallback map: rfq_quantize_act, rfq_fallback_map by
             scale threshold, rfq_gemm_phi
  mlp        a gated MLP block: rfq_quantize_act, rfq_gemm_swiglu_quantize,
             rfq_gemm (the down product)
  hif4       one linear layer in HiF4: rfq_hif4_quantize, rfq_hif4_gemm

Sizes: M activation rows (1 row of decode up to the 32768 rows of a video
transformer's sequence), K reduction columns, N outputs (mlp: N hidden units,
K in and out).  4096, 5120, 12288 and 13824 are the weight sizes of this
package's workloads; the others are generic layer sizes that do not divide by
the products' tiles.
"""
import math

import torch

import paper_2608_26581_amd as rfq

# A primary scale byte of 129 marks blocks whose largest magnitude is 16 or
# more: with N(0, 1) activations, tiles that hold an outlier channel.
PHI_THRESHOLD = 129


def listed():
    return [
        # Decode of one sequence, up projection: the smallest call there is.
        _case("decode_1_stream", "stream", 1, 12288, 4096),
        # Decode of a batch, down projection (long K, few outputs).
        _case("decode_16_down", "linear", 16, 4096, 12288, split=True),
        # Decode of a small batch through a layer whose K does not divide by
        # the kernels' 512-column groups.
        _case("decode_6_ragged", "linear", 6, 4096, 11008, split=True),
        # A short prompt through a gated MLP block.
        _case("prefill_200_mlp", "mlp", 200, 12288, 4096, split=True),
        # A prompt through a layer of awkward sizes, fp32 in and out.
        _case("prefill_1000_ragged", "linear", 1000, 5000, 2912, x="f32", z="f32"),
        # The activation quantizer by itself on a batch of tokens.
        _case("quantize_8192", "quantize", 8192, 0, 4096),
        # One quantization-aware training forward of a 4096-token batch.
        _case("qat_4096", "qat", 4096, 12288, 4096),
        # The same layer at inference with the fallback map.
        _case("phi_4096", "phi", 4096, 12288, 4096),
        # A video transformer's layer over a whole sequence: the largest call.
        _case("video_32768", "linear", 32768, 13824, 5120),
        # HiF4: decode of a few sequences.
        _case("hif4_decode_4", "hif4", 4, 12288, 4096, split=True),
        # HiF4: a short prompt, down projection.
        _case("hif4_prefill_300", "hif4", 300, 5120, 13824, split=True),
        # HiF4: a 4096-token batch.
        _case("hif4_4096", "hif4", 4096, 12288, 4096, split=True),
    ]


def _case(name, path, M, N, K, x="bf16", z="bf16", residual=True, split=False):
    return {"name": name, "path": path, "M": M, "N": N, "K": K, "x": x, "z": z,
            "residual": residual, "split": split}


def draw(rng):
    """One more case: a path, sizes spread over their logarithms (half of the
    K multiples of 512, the others any multiple of the block), both
    activation types and both output types, a few without the residual."""
    path = rng.choice(["quantize", "linear", "linear", "linear", "stream", "qat", "phi", "mlp",
                       "hif4", "hif4", "hif4"])

    def spread(lo, hi):
        return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))

    while True:
        M = spread(1, {"stream": 64, "qat": 8192, "phi": 8192, "mlp": 4096,
                       "hif4": 6000}.get(path, 32768))
        N = spread(1024, 16384)
        N = N if rng.random() < 0.25 else (N + 31) // 32 * 32
        K = spread(1024, 16384)
        block = 64 if path == "hif4" else 32
        whole = path in ("stream", "mlp") or rng.random() < 0.5
        K = max(1024, K // 512 * 512) if whole else K // block * block
        if path == "mlp":
            N = (N + 31) // 32 * 32
        if path == "quantize":
            N = 0
        work = M * max(N, 1) * K * (3 if path == "mlp" else 1)
        if path == "hif4":
            work *= 5
        if work <= 32768 * 13824 * 5120 // 2 and M * K <= 1 << 28:
            break
    small = M * max(N, 1) <= 1 << 25
    return {"path": path, "M": M, "N": N, "K": K,
            "x": "f32" if path != "mlp" and small and rng.random() < 0.25 else "bf16",
            "z": "f32" if path != "mlp" and small and rng.random() < 0.25 else "bf16",
            "residual": path == "phi" or rng.random() < 0.85,
            "split": path in ("linear", "hif4", "mlp") and rng.random() < 0.7}


# ---- inputs

_X = {"bf16": torch.bfloat16, "f32": torch.float32}


def _activations(M, K, dtype, gen):
    """N(0, 1) with 0.5% of the channels 50 times larger."""
    x = torch.randn(M, K, device="cuda", generator=gen)
    outliers = torch.randperm(K, device="cuda", generator=gen)[:max(1, round(0.005 * K))]
    x[:, outliers] *= 50.0
    return x.to(dtype)


def _weight(N, K, gen):
    return torch.randn(N, K, device="cuda", generator=gen) * 0.02


def _inputs(case, seed):
    """x and the fp32 master weights, from the seed alone."""
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    M, N, K = case["M"], case["N"], case["K"]
    x = _activations(M, K, _X[case["x"]], gen)
    if case["path"] == "quantize":
        return x, []
    if case["path"] == "mlp":
        return x, [_weight(N, K, gen), _weight(N, K, gen), _weight(K, N, gen)]
    return x, [_weight(N, K, gen)]


def prepare(case, seed):
    x, weights = _inputs(case, seed)
    state = {"case": case, "x": x}
    path = case["path"]
    if path == "qat":
        state["master"] = weights[0]
    elif path == "mlp":
        gate, up, down = weights
        state["gate_up"] = rfq.rfq_quantize_weight(rfq.interleave_gate_up(gate, up))
        state["down"] = rfq.rfq_quantize_weight(down)
    elif path == "hif4":
        state["w"] = rfq.rfq_hif4_quantize(weights[0], residual=False)[:2]
    elif path != "quantize":
        state["w"] = rfq.rfq_quantize_weight(weights[0])
    return state


# ---- one pass

def run(state):
    case, x = state["case"], state["x"]
    path, residual, z_dtype = case["path"], case["residual"], _X[case["z"]]
    if path == "quantize":
        return rfq.rfq_quantize_act(x, residual=residual)
    if path == "stream":
        return rfq.rfq_gemm_stream(x, *state["w"], residual=residual, out_dtype=z_dtype)
    if path == "hif4":
        q = rfq.rfq_hif4_quantize(x, residual=residual)
        return rfq.rfq_hif4_gemm(*q, *state["w"], out_dtype=z_dtype, split=case["split"])
    if path == "qat":
        w = rfq.rfq_quantize_weight(state["master"])
        q = rfq.rfq_quantize_act(x, residual=residual)
        return rfq.rfq_gemm(*q, *w, out_dtype=z_dtype), w
    q = rfq.rfq_quantize_act(x, residual=residual)
    if path == "phi":
        phi = rfq.rfq_fallback_map(q[2], q[1], rfq.RFQ_PHI_SCALE_AT_LEAST, PHI_THRESHOLD)
        return rfq.rfq_gemm_phi(*q, *state["w"], phi, out_dtype=z_dtype), phi
    if path == "mlp":
        h = rfq.rfq_gemm_swiglu_quantize(*q, *state["gate_up"], residual=residual)
        return rfq.rfq_gemm(*h[:4], *state["down"], out_dtype=z_dtype, split=case["split"])
    return rfq.rfq_gemm(*q, *state["w"], out_dtype=z_dtype, split=case["split"])


# ---- what a pass cannot do without

def work(case):
    """Bytes: each input of the pass read once, each output written once.
    Flops: both contractions of every product (the residual's is work that the
    method asks for)."""
    M, N, K = case["M"], case["N"], case["K"]
    path, terms = case["path"], 2 if case["residual"] else 1
    xb, zb = {"bf16": 2, "f32": 4}[case["x"]], {"bf16": 2, "f32": 4}[case["z"]]
    mx = 0.5 + 1 / 32
    if path == "quantize":
        return {"bytes": M * K * (xb + terms * mx), "flops": 0}
    if path == "mlp":
        return {"bytes": M * K * (xb + zb) + 3 * N * K * mx, "flops": 2 * terms * 3 * M * N * K}
    wb = 0.5 + 4 / 64 if path == "hif4" else (4 + mx if path == "qat" else mx)
    return {"bytes": M * K * xb + N * K * wb + M * N * zb, "flops": 2 * terms * M * N * K}


def tolerance(case):
    """Codes and maps are exact.  Products accumulate in fp32 in an order of
    their own: two such sums differ by up to a few 1e-7 (none at many sizes,
    where every partial sum fits 24 bits), and a bf16 result then by one
    rounding step (2^-8 of its value) where a sum lies that close to a
    rounding boundary: 2.4e-5 of the norm was measured between the split and
    unsplit products.  In the MLP block such steps in g, u and h also move
    codes of h: 2.4e-4 measured against 64-bit sums."""
    path = case["path"]
    if path == "quantize":
        return "exact"
    if path == "mlp":
        return {"rel": 1e-3, "max": 0.03}
    if case["z"] == "bf16":
        return {"rel": 1e-4, "max": 0.01}
    return {"rel": 1e-6, "max": 2e-5}


# ---- the same values in 64 bits

def _pow2(e):
    """2^e in float64, exact (e an integer tensor)."""
    return ((e.long() + 1023) << 52).view(torch.float64)


def _mxfp4(x):
    """The values of x's MXFP4 codes (and the block exponents) in float64."""
    b = x.double().reshape(x.shape[0], -1, 32)
    amax = b.abs().amax(-1, keepdim=True)
    e = torch.frexp(amax).exponent - 3                  # floor(log2 amax) - 2
    e = torch.where(amax == 0, torch.full_like(e, -127), e.clamp(-127, 127))
    y = b * _pow2(-e)
    a = y.abs()
    # Grid step 0.5 below 2, 1 below 4, 2 above; ties to the even code.
    step = torch.where(a < 2, 0.5, torch.where(a < 4, 1.0, 2.0)).to(a.dtype)
    q = (torch.round(a / step) * step).clamp(max=6.0)
    return (torch.copysign(q, y) * _pow2(e)).reshape(x.shape), e.squeeze(-1)


def _hif4(x):
    """The values of x's HiF4 codes in float64: the smallest macro scale S with
    7 S >= the block maximum, per 4 elements the smallest exponent that the
    8-element bit allows, quarters of the scale rounded to nearest even."""
    b = x.double().reshape(x.shape[0], -1, 64)
    byte = torch.arange(256, device=x.device)
    macro = (1.0 + (byte & 3).double() / 4) * _pow2((byte >> 2) - 48)
    amax = b.abs().amax(-1)
    S = macro[torch.searchsorted(7 * macro, amax.contiguous()).clamp(max=255)][..., None]
    g = b.reshape(*b.shape[:2], 16, 4).abs().amax(-1)
    need = (g > 1.75 * S).int() + (g > 3.5 * S).int()
    e8 = (need.reshape(*need.shape[:2], 8, 2) == 2).any(-1, keepdim=True).int()
    e16 = (need.reshape(*need.shape[:2], 8, 2) - e8).clamp(min=0)
    e = (e8 + e16).reshape(need.shape).repeat_interleave(4, -1)
    unit = S / 4 * _pow2(e)
    k = torch.round(b.abs() / unit).clamp(max=7)
    return torch.copysign(k * unit, b).reshape(x.shape)


def _with_residual(x, quantize, residual):
    q = quantize(x.double())
    return q + quantize(x.double() - q) if residual else q


def exact(case, seed):
    path, residual = case["path"], case["residual"]
    if path == "quantize":
        return None                                     # codes: nothing to compute in 64 bits
    x, weights = _inputs(case, seed)
    values = _hif4 if path == "hif4" else (lambda t: _mxfp4(t)[0])
    if path == "phi":
        q, e = _mxfp4(x.double())
        r = values(x.double() - q)
        M, K = x.shape
        rows, cols = -(-M // 64), -(-K // 256)
        marks = torch.zeros(rows * 64, cols * 8, dtype=torch.bool, device=x.device)
        marks[:M, :K // 32] = e + 127 >= PHI_THRESHOLD
        phi = marks.reshape(rows, 64, cols, 8).any(3).any(1)
        r *= phi.repeat_interleave(64, 0)[:M].repeat_interleave(256, 1)[:, :K]
        return (q + r) @ values(weights[0]).T, None
    xq = _with_residual(x, values, residual)
    if path == "mlp":
        g, u = ((xq @ values(w).T).bfloat16().double() for w in weights[:2])
        h = (g / (1 + torch.exp(-g)) * u).bfloat16()
        return _with_residual(h, values, residual) @ values(weights[2]).T
    z = xq @ values(weights[0]).T
    return (z, None) if path == "qat" else z
