"""Drop-in linear layer over the C ABI: forward and backward of Algorithm 1 as one autograd function.

Argument marshalling only, and that in native code: every arithmetic step runs in the library's kernels
(quartet_linear_fwd / quartet_linear_bwd).  torch provides device memory, streams and the autograd
graph.  There is no fallback: without a GPU or without the built library these calls raise.

Shapes: the flattened token count, in_features and out_features must be multiples of the Hadamard
block (32, the MXFP4 group, unless a layer asks for 64, 128 or 256).
"""
import torch

from . import binding as q
from . import _nn_native as _native          # fails loudly if it has not been built (python -m paper_2505_14669_amd.build)

_native.set_error(q.QuartetError)


class _PythonFunction(torch.autograd.Function):
    """The node's twin in Python over the same two native halves, for the calls that the native node does not serve (it says which):
    what torch does with an autograd function there, or the reason why it cannot, comes from torch itself."""

    @staticmethod
    def forward(ctx, x, weight, seed, rounding, hadamard_block):
        y, context = _native.forward(x, weight, hadamard_block)
        ctx.save_for_backward(context)
        ctx.call = (tuple(x.shape), weight.shape[0], seed, rounding, hadamard_block)
        return y

    @staticmethod
    def backward(ctx, dy):
        return (*_native.backward(*ctx.saved_tensors, dy, *ctx.call), None, None, None)


class QuartetLinearFunction:
    """y = x W^T with MXFP4 operands (Algorithm 1 Forward); the backward pass returns the gradients of
    Algorithm 1 Backward.  x: [..., in] bf16, weight: [out, in] bf16, seed: python int naming the
    stochastic-rounding draws of this call's backward pass, rounding: 0 stochastic / 1 nearest,
    hadamard_block: 32 (the method), 64, 128 or 256.  The autograd node is native code (csrc/nn_autograd.cpp)."""

    @staticmethod
    def apply(x, weight, seed, rounding, hadamard_block=32):
        call = (x, weight, int(seed), int(rounding), int(hadamard_block))
        y = _native.linear(*call)
        return _PythonFunction.apply(*call) if y is None else y


class QuartetLinear(torch.nn.Module):
    """nn.Linear replacement: weight [out, in] (bf16, or fp32 master weights cast to bf16 on the way
    in), optional bf16 bias added outside the quantized product.  Every backward pass uses a fresh stochastic-rounding seed: base seed, layer id and a
    per-layer call counter packed into 64 bits, so runs are reproducible and no two calls share draws."""
    _next_id = 0

    def __init__(self, in_features, out_features, bias=False, seed=0, rounding=0, device="cuda",
                 weight_dtype=torch.bfloat16, hadamard_block=32):
        super().__init__()
        self.hadamard_block = hadamard_block
        self.in_features, self.out_features = in_features, out_features
        w = torch.randn(out_features, in_features, device=device) * (in_features ** -0.5)
        # weight_dtype=torch.float32 keeps fp32 master weights; the kernels always see a bf16 copy
        self.weight = torch.nn.Parameter(w.to(weight_dtype))
        self.bias = torch.nn.Parameter(torch.zeros(out_features, dtype=torch.bfloat16, device=device)) if bias else None
        self.rounding = rounding
        self.base_seed = int(seed) & 0xFFFF
        self.layer_id = QuartetLinear._next_id & 0xFFFF
        QuartetLinear._next_id += 1
        self.calls = 0

    def forward(self, x):
        seed = (self.base_seed << 48) | (self.layer_id << 32) | (self.calls & 0xFFFFFFFF)
        self.calls += 1
        y = QuartetLinearFunction.apply(x, self.weight.to(torch.bfloat16), seed, self.rounding, self.hadamard_block)
        return y if self.bias is None else y + self.bias
