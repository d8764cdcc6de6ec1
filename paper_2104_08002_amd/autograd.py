"""The layer as a ``torch.autograd.Function`` and an ``nn.Module`` on top of the C-ABI binding.

Glue only: every arithmetic step of the three passes and of the bias and ReLU around them runs in the library's kernels;
torch supplies device memory, the stream and the autograd graph.  This is the interface the
paper's single-layer measurements use (Section 4.3: ``net.forward(x)`` and ``out.sum().backward()``).
"""
from __future__ import annotations

import torch
from torch.autograd import forward_ad

from . import binding


def _has_tangent(t) -> bool:
    # (unpack_dual asks for the level first too, but takes 2 us of a backward to say that there is none)
    return getattr(forward_ad, "_current_level", 0) >= 0 and forward_ad.unpack_dual(t).tangent is not None


class Conv1dFunction(torch.autograd.Function):
    """y = conv1d(x, w[, bias]) with dilation and zero padding; backward = one conv1d_bwd call."""

    @staticmethod
    def forward(ctx, x, w, bias, dilation: int, padding: int, relu: bool, bf16_out: bool):
        x, w = x.contiguous(), w.contiguous()
        ctx.save_for_backward(x, w)
        ctx.geometry = (int(dilation), int(padding))
        ctx.has_bias = bias is not None
        fused = bias is not None or relu or bf16_out
        if fused:
            y = binding.conv1d_fwd_ex(x, w, dilation, padding, bias=None if bias is None else bias.contiguous().float(),
                                      relu=relu, out_bf16=bf16_out)
        else:
            y = binding.conv1d_fwd(x, w, dilation, padding)
        ctx.relu = relu
        if relu and any(ctx.needs_input_grad):
            # not y itself: what follows the layer may change it in place
            ctx.y_positive = binding.conv1d_relu_mask(y)
        return y

    @staticmethod
    def backward(ctx, gy):
        x, w = ctx.saved_tensors
        d, P = ctx.geometry
        positive = ctx.y_positive if ctx.relu else None
        # create_graph or forward mode over this pass: the bias gradient is differentiable in gy
        if (gy.requires_grad and torch.is_grad_enabled()) or _has_tangent(gy):
            dy = gy
            if positive is not None:
                bit = torch.arange(8, dtype=torch.uint8, device=gy.device)
                dy = gy * ((positive[:, None] >> bit) & 1).bool().flatten()[:gy.numel()].view(gy.shape)
            gb = dy.float().sum(dim=(0, 2)) if ctx.has_bias else None
            dx, dw = binding.conv1d_bwd_ex(x, dy.to(x.dtype).contiguous(), w, d, P, out_bf16=x.dtype == torch.bfloat16)
        else:
            dx, dw, gb = binding.conv1d_layer_bwd(gy.resolve_neg().contiguous(), positive, x, w, d, P, ctx.has_bias)
        return dx, dw.to(w.dtype), gb, None, None, None, None


def conv1d(x, w, bias=None, dilation: int = 1, padding: int = 0, relu: bool = False, bf16_out: bool = False):
    return Conv1dFunction.apply(x, w, bias, dilation, padding, relu, bf16_out)


class Conv1d(torch.nn.Module):
    """Drop-in for ``torch.nn.Conv1d(C, K, S, dilation=d, padding=P)`` (stride 1, one group) on one MI355X."""

    def __init__(self, in_channels: int, out_channels: int, kernel_size: int, dilation: int = 1, padding: int = 0,
                 bias: bool = False, relu: bool = False, dtype=torch.float32, device="cuda"):
        super().__init__()
        self.dilation, self.padding, self.relu = dilation, padding, relu
        w = torch.empty(out_channels, in_channels, kernel_size, dtype=torch.float32, device=device)
        torch.nn.init.normal_(w, std=(in_channels * kernel_size) ** -0.5)
        self.weight = torch.nn.Parameter(w.to(dtype))
        self.bias = torch.nn.Parameter(torch.zeros(out_channels, dtype=torch.float32, device=device)) if bias else None

    def forward(self, x):
        return conv1d(x, self.weight, self.bias, self.dilation, self.padding, self.relu,
                      bf16_out=False)
