"""torch.autograd.Function over the resolve: forward bins and renders in one pass over the binned stream (coefficients and
accumulation kept for the gradient); backward runs the gradient kernel (wt_backward) for alpha and rgb. Depth receives
no gradient."""
from __future__ import annotations

import torch

from . import wt as _wt


class WaveletComposite(torch.autograd.Function):
    """out = WaveletComposite.apply(pixel, depth, alpha, rgb, spec, bg[, workspace])."""

    @staticmethod
    def forward(ctx, pixel, depth, alpha, rgb, spec: _wt.FrameSpec, bg, ws: _wt.Workspace = None):
        frags = _wt.Fragments(pixel, depth.detach(), alpha.detach().contiguous(), rgb.detach().contiguous())
        if ws is None:
            ws = _wt.Workspace(spec, frags.count, device=pixel.device)
        dev = pixel.device
        coeffs = torch.empty(spec.coeff_shape(), dtype=_wt.TORCH_DTYPES[spec.dtype], device=dev)
        accum = torch.empty((spec.pixels, spec.accum_width), dtype=torch.float32, device=dev)
        out = torch.empty((spec.pixels, 3), dtype=torch.float32, device=dev)
        _wt.render_accum(spec, frags, bg, ws, out, coeffs, accum)
        ctx.save_for_backward(pixel, frags.depth, frags.alpha, frags.rgb, coeffs, accum)
        ctx.spec, ctx.bg, ctx.ws = spec, tuple(float(b) for b in bg), ws
        return out

    @staticmethod
    def backward(ctx, grad_out):
        pixel, depth, alpha, rgb, coeffs, accum = ctx.saved_tensors
        frags = _wt.Fragments(pixel, depth, alpha, rgb)
        ga, gr = _wt.backward(ctx.spec, frags, coeffs, accum, ctx.bg, grad_out.contiguous().float(), ctx.ws)
        need = ctx.needs_input_grad
        return None, None, (ga if need[2] else None), (gr if need[3] else None), None, None, None


def composite(pixel, depth, alpha, rgb, spec, bg, ws=None):
    return WaveletComposite.apply(pixel, depth, alpha, rgb, spec, bg, ws)
