"""Performance cases of the library: what its users call, through the public entry points, over the sizes they call it with.

Kinds of a case
  layer    one linear layer of a training step through the C ABI's binding: quartet_linear_fwd + quartet_linear_bwd
           (the *_block twins for Hadamard blocks above 32), buffers and workspace the caller's own
  nn       the same step through nn.QuartetLinear and autograd, as a torch training loop runs it
  forward  quartet_linear_fwd alone (evaluation): any number of tokens, the saved context is part of the result
  infer    serving: weights quantized once, every call quantizes its activations and multiplies
  quant    one quantizer on one matrix (rows: groups along a row; transposed: groups along a column)
"""
import math

import torch

from paper_2505_14669_amd import binding as q
from paper_2505_14669_amd import nn as qnn

DEVICE = "cuda:0"
MAX_WORK = 16384 * 4096 * 11008      # tokens * in * out of the largest layer


def listed():
    return [
        # The smallest layer of a training step: four dependent launches of a few microseconds each, latency decides.
        dict(name="layer_256x512x512", kind="layer", tokens=256, inf=512, outf=512, block=32, rounding=0, bf16=False),
        # A small model's layer in a torch training loop, no size a multiple of a tile: autograd, allocations and launches.
        dict(name="nn_288x320x352", kind="nn", tokens=288, inf=320, outf=352, block=32, rounding=1),
        # Serving, a decode batch of a few tokens against a 7B-shaped gate projection: reads the 4-bit weights once.
        dict(name="infer_24x4096x11008", kind="infer", tokens=24, inf=4096, outf=11008, bf16=True),
        # Evaluation of an MLP layer on a ragged number of tokens: both operands quantized, one product.
        dict(name="forward_1003x2048x5632", kind="forward", tokens=1003, inf=2048, outf=5632, bf16=True),
        # Attention projection (Q/K/V/O) of a 2048-wide model: one round of tiles.
        dict(name="layer_4096x2048x2048", kind="layer", tokens=4096, inf=2048, outf=2048, block=32, rounding=0, bf16=False),
        # A layer whose sizes are multiples of 32 and of nothing larger, nearest rounding, bf16 gradients.
        dict(name="layer_2336x1376x3168", kind="layer", tokens=2336, inf=1376, outf=3168, block=32, rounding=1, bf16=True),
        # MLP down projection of a 2048-wide model in a torch training loop.
        dict(name="nn_8192x5632x2048", kind="nn", tokens=8192, inf=5632, outf=2048, block=32, rounding=0),
        # Attention projection of a 7B-shaped block.
        dict(name="layer_16384x4096x4096", kind="layer", tokens=16384, inf=4096, outf=4096, block=32, rounding=0, bf16=False),
        # MLP gate / up projection of a 7B-shaped block: the largest layer.
        dict(name="layer_16384x4096x11008", kind="layer", tokens=16384, inf=4096, outf=11008, block=32, rounding=0, bf16=False),
        # Hadamard block of 128 elements on an attention projection.
        dict(name="block128_4096x2048x2048", kind="layer", tokens=4096, inf=2048, outf=2048, block=128, rounding=0, bf16=False),
        # Hadamard block of 256 elements (the widest the method prices) on an MLP up projection, torch training loop.
        dict(name="block256_8192x2048x5632", kind="nn", tokens=8192, inf=2048, outf=5632, block=256, rounding=0),
        # The quantizer alone: a full-size gradient transposed with stochastic rounding.
        dict(name="quant_sr_t_16384x11008", kind="quant", rows=16384, cols=11008, mode="sr", transpose=True),
    ]


def _log_size(rng, low, high, step):
    """A multiple of step in [low, high], uniform over the logarithm."""
    v = int(round(math.exp(rng.uniform(math.log(low), math.log(high))) / step)) * step
    return min(max(v, -(-low // step) * step), high // step * step)


def draw(rng):
    kind = rng.choices(["layer", "nn", "infer", "forward", "quant"], [4, 2, 2, 1, 2])[0]
    if kind == "quant":
        return dict(kind=kind, rows=_log_size(rng, 256, 16384, 32), cols=_log_size(rng, 256, 11008, 32),
                    mode=rng.choice(["fwd", "rtn", "sr"]), transpose=rng.random() < 0.5)
    if kind == "infer":
        # a quarter of the output widths is odd (a vocabulary, a fused head)
        outf = _log_size(rng, 256, 11008, 32) - (rng.randrange(1, 32) if rng.random() < 0.25 else 0)
        return dict(kind=kind, tokens=_log_size(rng, 1, 1024, 1), inf=_log_size(rng, 256, 11008, 32), outf=outf,
                    bf16=rng.random() < 0.75)
    if kind == "forward":
        return dict(kind=kind, tokens=_log_size(rng, 32, 8192, 1), inf=_log_size(rng, 256, 5632, 32),
                    outf=_log_size(rng, 256, 5632, 32), bf16=rng.random() < 0.5)
    block = rng.choices([32, 64, 128, 256], [8, 1, 1, 1])[0]
    while True:
        tokens, inf, outf = (_log_size(rng, 256, high, block) for high in (16384, 11008, 11008))
        if tokens * inf * outf <= MAX_WORK:
            break
    case = dict(kind=kind, tokens=tokens, inf=inf, outf=outf, block=block, rounding=int(rng.random() < 0.4))
    if kind == "layer":
        case["bf16"] = rng.random() < 0.5
    return case


# ------------------------------------------------------------------ inputs: the value distributions of the benchmark

def _activations(g, rows, cols):
    """Student-t(3) rows of unit RMS with log-normal channel scales (heavy tails and outlier channels)."""
    x = torch.randn((rows, cols), generator=g, device=DEVICE)
    chi = torch.zeros((rows, cols), device=DEVICE)
    for _ in range(3):
        chi += torch.randn((rows, cols), generator=g, device=DEVICE).square_()
    x /= chi.div_(3.0).sqrt_()
    x /= x.square().mean(dim=1, keepdim=True).sqrt_()
    x *= torch.exp(torch.randn((cols,), generator=g, device=DEVICE))[None, :]
    return x.to(torch.bfloat16)


def _normal(g, rows, cols, sigma):
    return torch.randn((rows, cols), generator=g, device=DEVICE).mul_(sigma).to(torch.bfloat16)


def _empty(shape, dtype):
    return torch.empty(shape, dtype=dtype, device=DEVICE)


class _Quantized:
    """Buffers of one MXFP4 tensor [rows x k] and its clipping mask."""

    def __init__(self, rows, k, with_mask=True):
        self.codes = _empty((rows, k // 2), torch.uint8)
        # bytes of the scale tiles that hold no group are never written: clear them once, as they come back with the result
        self.scales = torch.zeros((q.quartet_scale_bytes(rows, k),), dtype=torch.uint8, device=DEVICE)
        self.mask = _empty((rows, k // 32), torch.int32) if with_mask else None


class _State:
    def __init__(self, **kw):
        self.__dict__.update(kw)


def prepare(case, seed):
    g = torch.Generator(device=DEVICE)
    g.manual_seed(seed)
    kind = case["kind"]
    if kind == "quant":
        rows, cols = case["rows"], case["cols"]
        x = torch.randn((rows, cols), generator=g, device=DEVICE)
        x = torch.where(torch.rand((rows, cols), generator=g, device=DEVICE) < 0.001, x * 50.0, x).to(torch.bfloat16)
        out = _Quantized(cols, rows) if case["transpose"] else _Quantized(rows, cols)
        return _State(kind=kind, case=case, x=x, out=out, seed=seed, sign=q.quartet_sign_word(seed))
    t, i, o = case["tokens"], case["inf"], case["outf"]
    x, w = _activations(g, t, i), _normal(g, o, i, 0.02)
    if kind == "nn":
        layer = qnn.QuartetLinear(i, o, seed=seed, rounding=case["rounding"], hadamard_block=case["block"])
        layer.layer_id = 0           # as in a program that builds its model once: the draws depend on the seed alone
        with torch.no_grad():
            layer.weight.copy_(w)
        return _State(kind=kind, layer=layer, x=x.requires_grad_(True), dy=_normal(g, t, o, 1e-3))
    res = torch.bfloat16 if case["bf16"] else torch.float32
    dt = q.QUARTET_DTYPE_BF16 if case["bf16"] else q.QUARTET_DTYPE_F32
    s = _State(kind=kind, case=case, x=x, w=w, t=t, i=i, o=o, dt=dt, y=_empty((t, o), res), xq=_Quantized(t, i, kind != "infer"),
               wq=_Quantized(o, i))
    if kind == "infer":
        q.check(q.quartet_quant_fwd(w, o, i, i, 0, s.wq.codes, s.wq.scales, None))
    if kind == "layer":
        s.dy, s.seed, s.block, s.rounding = _normal(g, t, o, 1e-3), seed, case["block"], case["rounding"]
        s.dx, s.dw = _empty((t, i), res), _empty((o, i), res)
        s.ws_bytes = q.quartet_linear_workspace_bytes_block(t, i, o, s.block)
        s.ws = _empty((s.ws_bytes,), torch.uint8)
    return s


def run(s):
    if s.kind == "nn":
        s.x.grad = s.layer.weight.grad = None
        y = s.layer(s.x)
        y.backward(s.dy)
        return {"y": y.detach(), "dx": s.x.grad, "dw": s.layer.weight.grad}
    if s.kind == "quant":
        rows, cols = s.x.shape
        r, k = (cols, rows) if s.case["transpose"] else (rows, cols)
        if s.case["mode"] == "fwd":
            q.check(q.quartet_quant_fwd(s.x, r, k, cols, s.case["transpose"], s.out.codes, s.out.scales, s.out.mask))
            return {"codes": s.out.codes, "scales": s.out.scales, "mask": s.out.mask}
        rounding = q.QUARTET_ROUND_STOCHASTIC if s.case["mode"] == "sr" else q.QUARTET_ROUND_NEAREST
        q.check(q.quartet_quant_bwd_sr(s.x, r, k, cols, s.case["transpose"], s.sign, s.seed, 2, rounding, s.out.codes, s.out.scales))
        return {"codes": s.out.codes, "scales": s.out.scales}
    if s.kind == "infer":
        q.check(q.quartet_quant_fwd(s.x, s.t, s.i, s.i, 0, s.xq.codes, s.xq.scales, None))
        q.check(q.quartet_mxfp4_gemm(s.xq.codes, s.xq.scales, s.wq.codes, s.wq.scales, s.t, s.o, s.i, 1.0, s.y, s.dt, s.o))
        return {"y": s.y}
    if s.kind == "forward":
        q.check(q.quartet_linear_fwd(s.x, s.w, s.t, s.i, s.o, s.y, s.dt, s.xq.codes, s.xq.scales, s.xq.mask,
                                     s.wq.codes, s.wq.scales, s.wq.mask))
        return {"y": s.y, "xq_codes": s.xq.codes, "xq_scales": s.xq.scales, "x_mask": s.xq.mask,
                "wq_codes": s.wq.codes, "wq_scales": s.wq.scales, "w_mask": s.wq.mask}
    ctx = (s.xq.codes, s.xq.scales, s.xq.mask, s.wq.codes, s.wq.scales, s.wq.mask)
    if s.block == 32:
        q.check(q.quartet_linear_fwd(s.x, s.w, s.t, s.i, s.o, s.y, s.dt, *ctx))
        q.check(q.quartet_linear_bwd(s.dy, s.t, s.i, s.o, *ctx, s.seed, s.rounding, s.dx, s.dw, s.dt, s.ws, s.ws_bytes))
    else:
        q.check(q.quartet_linear_fwd_block(s.x, s.w, s.t, s.i, s.o, s.block, s.y, s.dt, *ctx))
        q.check(q.quartet_linear_bwd_block(s.dy, s.t, s.i, s.o, s.block, *ctx, s.seed, s.rounding, s.dx, s.dw, s.dt,
                                           s.ws, s.ws_bytes))
    return {"y": s.y, "dx": s.dx, "dw": s.dw}


def _mxfp4_bytes(n):
    return n * 17.0 / 32.0               # half a byte per code, one scale byte per 32


def work(case):
    """Compulsory work: every input read once, every result written once; two flops per multiply-add of the products."""
    kind = case["kind"]
    if kind == "quant":
        n = float(case["rows"]) * case["cols"]
        return {"bytes": 2 * n + _mxfp4_bytes(n) + (n / 8 if case["mode"] == "fwd" else 0), "flops": 10.0 * n}
    t, i, o = float(case["tokens"]), float(case["inf"]), float(case["outf"])
    res = 2.0 if case.get("bf16", True) else 4.0
    if kind == "infer":
        return {"bytes": 2 * t * i + _mxfp4_bytes(o * i) + res * t * o, "flops": 2 * t * i * o}
    context = _mxfp4_bytes(t * i + o * i) + (t * i + o * i) / 8
    forward = 2 * (t * i + o * i) + res * t * o
    if kind == "forward":
        return {"bytes": forward + context, "flops": 2 * t * i * o}
    return {"bytes": forward + 2 * t * o + res * (t * i + o * i), "flops": 6 * t * i * o}


def tolerance(case):
    # Codes, scales and masks are fixed bit for bit by the method.  The products of 4-bit values are exact; on these inputs
    # their fp32 sums are nearly always exact too (measured: three tile shapes, hence three orders of the sums, and fp64
    # give the same bits on eight of the listed cases), so what is left to another order is a last fp32 bit here and
    # there, and in a bf16 result the rounding of the few values that such a bit moves across a tie.
    if case["kind"] == "quant":
        return "exact"
    if case.get("bf16", True):
        return {"rel": 1e-4, "max": 0.01}
    return {"rel": 2.5e-7, "max": 2e-6}
