"""PyTorch operator over the C ABI, and a linear layer built on it.

``torch.ops.marlin_mi355x.gemm(A, w_packed, s_packed, K, N, group, sparse)``
is registered with ``torch.library.custom_op``, so code that dispatches
through ``torch.ops`` (a serving engine's quantised linear layer, for
instance; the paper integrates its kernel into vLLM this way, Section 5.2)
calls the HIP kernels as one opaque operator.  Its fake implementation gives
the output's shape, dtype and device for meta and fake tensors, without a
GPU.  The real implementation is ``ops.gemm``: argument checks, an output
allocation and one ``marlin_gemm`` (or ``marlin_gemm_sparse``) call on the
current stream.  There is no autograd formula (inference only).

``MarlinLinear`` holds one quantised, packed weight matrix and applies it to
the last dimension of its input, y = x W (no bias).  ``from_float`` takes an
``nn.Linear``-style fp16 weight [out_features, in_features] and quantises and
packs it on the GPU, in one launch where it is contiguous (``ops.quantize_linear``).

HIP graphs: the operator enqueues kernels only, so it can be captured.  Its
workspace is the per-(device, stream) one of ``ops.gemm``, allocated on first
use; call the layer once eagerly on the capturing stream before capturing so
that no allocation happens inside the capture.
"""
from __future__ import annotations

import torch

from . import ops

_NS = "marlin_mi355x"


@torch.library.custom_op(_NS + "::gemm", mutates_args=())
def gemm(A: torch.Tensor, w_packed: torch.Tensor, s_packed: torch.Tensor, K: int, N: int,
         group: int, sparse: bool = False) -> torch.Tensor:
    return ops.gemm(A, w_packed, s_packed, K, N, group=group, sparse=sparse)


@gemm.register_fake
def _gemm_fake(A, w_packed, s_packed, K, N, group, sparse=False):
    if A.dim() != 2 or A.shape[1] != K:
        raise ValueError("marlin_mi355x::gemm: A must be [M, K] with K=%d" % K)
    if A.dtype != torch.float16:
        raise TypeError("marlin_mi355x::gemm: A must be float16")
    return A.new_empty((A.shape[0], N))


# What the check below asks of torch, bound once: looking the names up took as
# long as asking.
_Tensor, _grad_enabled = torch.Tensor, torch.is_grad_enabled
_dispatch_modes, _function_modes = torch._C._len_torch_dispatch_stack, torch._C._len_torch_function_stack
_transforms, _tracing = torch._C._functorch.peek_interpreter_stack, torch._C._get_tracing_state
_forward_ad, _profiling = torch.autograd.forward_ad, torch.autograd._profiler_enabled


def _plain(x: torch.Tensor, w: torch.Tensor, s: torch.Tensor) -> bool:
    """Nothing but the CUDA implementation would see the operator's call on
    these three tensors: no tracing or compiling, no subclass, mode, transform,
    dual level or profiler, no gradient, no lazily negated view.  The layer then
    calls it directly: the operator's dispatch (5 us through Python, 28 -> 12 us
    a call with the above) is as long as a small decode GEMM.  (Where the
    buffers are is checked by the call itself; packed bytes have no sign.)"""
    return (not torch.compiler.is_compiling()
            and type(x) is _Tensor and type(w) is _Tensor and type(s) is _Tensor
            and x.is_cuda
            and not ((x.requires_grad or s.requires_grad) and _grad_enabled())
            and not x.is_neg() and not s.is_neg()
            and _dispatch_modes() == 0
            and _function_modes() == 0
            and _transforms() is None
            and _tracing() is None
            and _forward_ad._current_level < 0
            and not _profiling())


class MarlinLinear(torch.nn.Module):
    """y = x W with W quantised to 4 bits (zero point 8, fp16 group scales)."""

    def __init__(self, w_packed: torch.Tensor, s_packed: torch.Tensor, in_features: int,
                 out_features: int, group: int = 128, sparse: bool = False):
        super().__init__()
        self.in_features = int(in_features)
        self.out_features = int(out_features)
        self.group = ops._group(self.in_features, group)
        self.sparse = bool(sparse)
        self.register_buffer("w_packed", w_packed)
        self.register_buffer("s_packed", s_packed)

    @classmethod
    def from_float(cls, weight: torch.Tensor, group=128, ratios=ops.CLIP_RATIOS) -> "MarlinLinear":
        """weight: fp16 [out_features, in_features] on the GPU (nn.Linear layout)."""
        if weight.dim() != 2:
            raise ValueError("from_float: weight must be 2-D [out_features, in_features]")
        N, K = weight.shape
        wp, sp = ops.quantize_linear(weight, group=group, ratios=ratios)
        return cls(wp, sp, K, N, group)

    def forward(self, x: torch.Tensor) -> torch.Tensor:
        if x.shape[-1] != self.in_features:
            raise ValueError("MarlinLinear: last dimension %d, expected %d" % (x.shape[-1], self.in_features))
        w, s, K, N = self.w_packed, self.s_packed, self.in_features, self.out_features
        if _plain(x, w, s):
            if x.dim() == 2:
                return ops.gemm(x, w, s, K, N, self.group, sparse=self.sparse)
            y = ops.gemm(x.reshape(-1, K), w, s, K, N, self.group, sparse=self.sparse)
            return y.view(*x.shape[:-1], N)
        y = torch.ops.marlin_mi355x.gemm(x.reshape(-1, K), w, s, K, N, self.group, self.sparse)
        return y.reshape(*x.shape[:-1], N)

    def extra_repr(self) -> str:
        return "in_features=%d, out_features=%d, group=%d, sparse=%s" % (
            self.in_features, self.out_features, self.group, self.sparse)
