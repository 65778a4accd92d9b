"""torch.autograd binding of the renderer: forward = plx_render_fwd, backward
= plx_render_bwd (reverse replay with recomputed transmittance).  Saved are
the rays and, for a batch in ray order (plx_render_fwd_rays and
plx_render_bwd_rays), its rays' values and the first occupied samples of each,
else its optical depths and segment lists; nothing where no backward can
follow."""
from __future__ import annotations

import torch

from . import binding as B


def _aligned(t):
    """t, or a copy where a saved-tensor hook handed back memory that is not
    256-byte aligned, as the workspaces have to be."""
    return t if t.data_ptr() % 256 == 0 and t.is_contiguous() else t.clone(memory_format=torch.contiguous_format)


class RenderFn(torch.autograd.Function):
    """rgb = RenderFn.apply(params, grid, rays_o, rays_d, bg[, record]).

    ``params`` is the grid's FP32 record tensor [M, 32] (``grid.data`` for
    FP32 grids, ``grid.master`` for 16-bit ones); its gradient has the same
    record layout (slots 0..26 SH, slot 28 density).  The forward reads the
    grid's stored records.  record: whether a backward may follow (the
    caller's grad mode, which a forward does not see); without one, or where
    params need no gradient, no samples are kept."""

    @staticmethod
    def forward(ctx, params, grid, rays_o, rays_d, bg, record=True):
        n = rays_o.shape[0]
        rgb = torch.empty(n, 3, dtype=torch.float32, device=rays_o.device)
        desc = grid.desc()
        ctx.grid = grid
        ctx.bg = tuple(bg)
        if B.ray_order_grad(desc, n):
            ctx.bins = None
            if not (record and ctx.needs_input_grad[0]):
                B.plx_render_fwd_rays(desc, rays_o, rays_d, rgb, None, None, bg)
                return rgb
            # in ray order, keeping the occupied samples' values
            ctx.cap = B.ray_cap(n, desc)
            work = B.make_ray_work(n, device=rays_o.device, cap=ctx.cap)
            B.plx_render_fwd_rays(desc, rays_o, rays_d, rgb, None, work, bg)
            ctx.save_for_backward(rays_o, rays_d, work.ray_ws, work.samp_ws)
        else:
            tau = torch.empty(n, dtype=torch.float32, device=rays_o.device)
            ctx.bins = B.make_bins(desc, rays_o, rays_d)
            B.plx_render_fwd(desc, rays_o, rays_d, rgb, tau, bg, bins=ctx.bins)
            ctx.save_for_backward(rays_o, rays_d, tau)
        return rgb

    @staticmethod
    def backward(ctx, grad_rgb):
        rays_o, rays_d, *saved = ctx.saved_tensors
        g = ctx.grid
        grad = torch.zeros(g.n_vox, B.REC_SLOTS, dtype=torch.float32, device=rays_o.device)
        touched = torch.zeros(g.n_vox, dtype=torch.uint8, device=rays_o.device)
        grad_rgb = grad_rgb.contiguous().float()
        if ctx.bins is None:
            work = B.RayWork(rays_o.shape[0], *map(_aligned, saved), ctx.cap)
            B.plx_render_bwd_rays(g.desc(), rays_o, rays_d, grad_rgb, work, grad, touched, ctx.bg)
        else:
            B.plx_render_bwd(g.desc(), rays_o, rays_d, grad_rgb, saved[0], grad, touched, ctx.bg, bins=ctx.bins)
        return grad, None, None, None, None, None


def render(grid, rays_o, rays_d, bg=(1.0, 1.0, 1.0)) -> torch.Tensor:
    """Differentiable render of a ray batch with respect to the grid's FP32
    records (set ``grid.param_records().requires_grad_()`` first)."""
    return RenderFn.apply(grid.param_records(), grid, rays_o, rays_d, tuple(bg), torch.is_grad_enabled())
