"""ctypes binding of libplenoxel_hip.so (include/plenoxel.h).

Argument marshalling only: every function here checks tensor devices, dtypes,
shapes and contiguity, passes raw device pointers and the current HIP stream,
and raises ``PlxError`` with the library's message on a non-zero return.
All compute runs in the library's kernels.  The library is loaded from
``_build/`` next to this file; if it is missing, importing the functions
fails loudly (build it with ``python paper_2112_05131_amd/build.py``).
"""
from __future__ import annotations

import ctypes
from dataclasses import dataclass
import math
import os
import re

import torch

HERE = os.path.dirname(os.path.abspath(__file__))
ROOT = os.path.dirname(HERE)
LIB_PATH = os.path.join(HERE, "_build", "libplenoxel_hip.so")
HEADER = os.path.join(ROOT, "include", "plenoxel.h")

PLX_OK, PLX_EINVAL, PLX_EDEVICE, PLX_EUNSUPPORTED, PLX_ENOMEM = 0, 1, 2, 3, 4
COUNT_WORKSPACE_BYTES = 256
PLX_F32, PLX_BF16, PLX_F16 = 0, 1, 2
REC_SLOTS = 32
SLOT_SIGMA = 28
NSH = 27
DTYPES = {"f32": PLX_F32, "bf16": PLX_BF16, "f16": PLX_F16}


class PlxError(RuntimeError):
    def __init__(self, code, msg):
        super().__init__(f"[plx error {code}] {msg}")
        self.code = code


class PlxGrid(ctypes.Structure):
    _fields_ = [
        ("reso", ctypes.c_int32 * 3),
        ("scale", ctypes.c_float * 3),
        ("offset", ctypes.c_float * 3),
        ("step", ctypes.c_float),
        ("sh_dtype", ctypes.c_int32),
        ("n_vox", ctypes.c_int64),
        ("index", ctypes.c_void_p),
        ("data", ctypes.c_void_p),
        ("occ", ctypes.c_void_p),
    ]


class PlxRenderOpts(ctypes.Structure):
    _fields_ = [
        ("background", ctypes.c_float * 3),
        ("lambda_sparsity", ctypes.c_float),
        ("lambda_beta", ctypes.c_float),
        ("beta_eps", ctypes.c_float),
        ("reg_loss_sum", ctypes.c_void_p),
        ("background_rgb", ctypes.c_void_p),
        ("grad_background", ctypes.c_void_p),
        ("kernel_events", ctypes.c_void_p),
    ]


@dataclass
class Priors:
    """The optional sparsity (Cauchy) and beta priors of the gradient calls
    (plx_render_opts); `loss` is a device float64 tensor of 2 elements that
    gets (L_s, L_b) added, or None."""

    lambda_sparsity: float = 0.0
    lambda_beta: float = 0.0
    beta_eps: float = 1e-3
    loss: torch.Tensor | None = None


class PlxBins(ctypes.Structure):
    _fields_ = [
        ("n_rays", ctypes.c_int64),
        ("n_seg", ctypes.c_int64),
        ("n_samp", ctypes.c_int64),
        ("n_brick", ctypes.c_int64),
        ("ray_buf", ctypes.c_void_p),
        ("ray_buf_bytes", ctypes.c_int64),
        ("seg_buf", ctypes.c_void_p),
        ("seg_buf_bytes", ctypes.c_int64),
        ("samp_buf", ctypes.c_void_p),
        ("samp_buf_bytes", ctypes.c_int64),
    ]


class PlxView(ctypes.Structure):
    _fields_ = [
        ("c2w", ctypes.c_double * 12),
        ("focal", ctypes.c_double),
        ("width", ctypes.c_int32),
        ("height", ctypes.c_int32),
        ("scene", ctypes.c_int32),
        ("reserved", ctypes.c_int32),
        ("out_offset", ctypes.c_int64),
    ]


_lib = None
_P = ctypes.c_void_p
_I64 = ctypes.c_int64
_F = ctypes.c_float
_I32 = ctypes.c_int32
_GP = ctypes.POINTER(PlxGrid)
_OP = ctypes.POINTER(PlxRenderOpts)
_BP = ctypes.POINTER(PlxBins)

_SIGS = {
    "plx_last_error": ([], ctypes.c_char_p),
    "plx_version": ([], ctypes.c_char_p),
    "plx_record_bytes": ([_I32], _I64),
    "plx_occ_words": ([_P], _I64),
    "plx_occ_bytes": ([_P], _I64),
    "plx_occ_brick_offset": ([_P], _I64),
    "plx_grid_geometry": ([_P, _P, _P, ctypes.c_double, _P, _P, _P], ctypes.c_int),
    "plx_lr_schedule": ([ctypes.c_double] * 6, ctypes.c_double),
    "plx_grid_workspace_bytes": ([_P], _I64),
    "plx_mask_count": ([_P, _I64, _P, _I64, _P, _P], ctypes.c_int),
    "plx_grid_create": ([_P, _P, _P, _P, _I64, _P], ctypes.c_int),
    "plx_records_pack": ([_I32, _I64, _P, _P, _F, _F, _P, _P], ctypes.c_int),
    "plx_records_unpack": ([_I32, _I64, _P, _P, _P, _P], ctypes.c_int),
    "plx_records_convert": ([_I32, _P, _I32, _P, _I64, _P], ctypes.c_int),
    "plx_grid_build_occupancy": ([_GP, _P, _P], ctypes.c_int),
    "plx_grid_prune_count": ([_GP, _F, _P, _P, _I64, _P, _P, _P], ctypes.c_int),
    "plx_grid_prune_weight_count": ([_GP, _P, _F, _P, _P, _I64, _P, _P, _P], ctypes.c_int),
    "plx_grid_prune_apply": ([_GP, _P, _GP, _P, _I64, _P], ctypes.c_int),
    "plx_grid_upsample_count": ([_GP, _P, _P, _I64, _P, _P], ctypes.c_int),
    "plx_grid_upsample_apply": ([_GP, _GP, _P, _I64, _P], ctypes.c_int),
    "plx_rays_to_ndc": ([_P, _P, _I64, _I32, _I32, ctypes.c_double, ctypes.c_double, _P, _P, _P],
                        ctypes.c_int),
    "plx_bg_tv_grad": ([_GP, _I64, _I64, _F, _F, _F, _P, _P, _P, _P], ctypes.c_int),
    "plx_bg_render_fwd": ([_GP, _P, _P, _I64, _P, _P, _P, _P], ctypes.c_int),
    "plx_bg_render_bwd": ([_GP, _P, _P, _I64, _P, _P, _P, _P, _P], ctypes.c_int),
    "plx_bins_ray_bytes": ([_P, _I64], _I64),
    "plx_bins_seg_bytes": ([_I64], _I64),
    "plx_bins_samp_bytes": ([_I64, _I64], _I64),
    "plx_bins_count": ([_GP, _P, _P, _I64, _P, _I64, _P, _P], ctypes.c_int),
    "plx_bins_apply": ([_GP, _P, _P, _BP, _P], ctypes.c_int),
    "plx_bins_verify": ([_GP, _BP, _P], ctypes.c_int),
    "plx_render_fwd": ([_GP, _OP, _P, _P, _I64, _BP, _P, _P, _P], ctypes.c_int),
    "plx_render_bwd": ([_GP, _OP, _P, _P, _I64, _BP, _P, _P, _P, _P, _P], ctypes.c_int),
    "plx_render_train": ([_GP, _OP, _P, _P, _P, _I64, _BP, _F, _P, _P, _P, _P, _P], ctypes.c_int),
    "plx_render_fwd_rays": ([_GP, _OP, _P, _P, _I64, _P, _P, _P, _I64, _P, _I64, _I32, _P], ctypes.c_int),
    "plx_render_bwd_rays": ([_GP, _OP, _P, _P, _I64, _P, _P, _I64, _P, _I64, _I32, _P, _P, _P], ctypes.c_int),
    "plx_rays_ray_bytes": ([_I64], _I64),
    "plx_rays_samp_bytes": ([_I64, _I32], _I64),
    "plx_render_train_rays": ([_GP, _OP, _P, _P, _P, _I64, _P, _I64, _P, _I64, _I32, _F, _P, _P, _P, _P, _P],
                              ctypes.c_int),
    "plx_render_max_weight": ([_GP, _P, _P, _I64, _BP, _P, _P], ctypes.c_int),
    "plx_render_train_static": ([_GP, _OP, _P, _P, _P, _I64, _F, _P, _P, _P, _P, _P], ctypes.c_int),
    "plx_render_state_bytes": ([_I64, _I32], _I64),
    "plx_render_fwd_state": ([_GP, _OP, _P, _P, _I64, _P, _P, _P, _I64, _I32, _P], ctypes.c_int),
    "plx_render_bwd_state": ([_GP, _OP, _P, _P, _I64, _P, _P, _P, _I64, _I32, _P, _P, _P],
                             ctypes.c_int),
    "plx_render_stats": ([_GP, _P, _P, _I64, _P, _P, _P, _I64, _P, _P], ctypes.c_int),
    "plx_scene_table_bytes": ([_I32], _I64),
    "plx_scene_table_set": ([_GP, _I32, _P, _I64, _P], ctypes.c_int),
    "plx_render_views": ([_P, _I32, _I32, _P, _I32, _OP, _P, _P, _P], ctypes.c_int),
    "plx_render_views_status": ([_P, _P], ctypes.c_int),
    "plx_tv_grad": ([_GP, _I64, _I64, _F, _F, _F, _P, _P, _P, _P], ctypes.c_int),
    "plx_touched_count": ([_P, _I64, _P, _I64, _P, _P], ctypes.c_int),
    "plx_rmsprop_step": ([_GP, _P, _P, _P, _P, _F, _F, _F, _F, _P], ctypes.c_int),
}


def header_functions() -> list[str]:
    """Names of the functions declared in include/plenoxel.h."""
    text = open(HEADER).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(plx_[a-z0-9_]+)\s*\(", text)))


def lib():
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise RuntimeError(
                f"HIP library not built: {LIB_PATH} is missing "
                "(run python paper_2112_05131_amd/build.py)")
        L = ctypes.CDLL(LIB_PATH)
        for name, (args, res) in _SIGS.items():
            fn = getattr(L, name)
            fn.argtypes = args
            fn.restype = res
        _lib = L
    return _lib


def _check(rc):
    if rc != PLX_OK:
        msg = lib().plx_last_error().decode(errors="replace")
        raise PlxError(rc, msg)


def _stream():
    return ctypes.c_void_p(torch.cuda.current_stream().cuda_stream)


def _dptr(t: torch.Tensor | None, name: str, dtype=None, numel=None, device_ok=True):
    if t is None:
        return None
    if not t.is_cuda:
        raise ValueError(f"{name} must be a device tensor")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")
    if dtype is not None and t.dtype != dtype:
        raise ValueError(f"{name} must be {dtype}, got {t.dtype}")
    if numel is not None and t.numel() != numel:
        raise ValueError(f"{name} must have {numel} elements, got {t.numel()}")
    return ctypes.c_void_p(t.data_ptr())


def _i3(v):
    return (ctypes.c_int32 * 3)(*[int(x) for x in v])


def workspace(nbytes: int, device=None) -> torch.Tensor:
    """A device buffer for a call's workspace argument (torch allocations
    are 256-byte aligned)."""
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8,
                       device=device if device is not None else "cuda")


def _ws(ws, nbytes: int, device=None):
    """(pointer, bytes) of a given workspace tensor, or of a new one."""
    if ws is None:
        ws = workspace(nbytes, device)
    return _dptr(ws, "ws", torch.uint8), ws.numel(), ws


# --------------------------------------------------------------------- misc

def plx_version() -> str:
    return lib().plx_version().decode()


def plx_record_bytes(sh_dtype: int) -> int:
    return int(lib().plx_record_bytes(sh_dtype))


def plx_occ_words(reso) -> int:
    return int(lib().plx_occ_words(ctypes.cast(_i3(reso), _P)))


def plx_occ_bytes(reso) -> int:
    return int(lib().plx_occ_bytes(ctypes.cast(_i3(reso), _P)))


def plx_occ_brick_offset(reso) -> int:
    return int(lib().plx_occ_brick_offset(ctypes.cast(_i3(reso), _P)))


def plx_grid_geometry(reso, lo=(-0.5,) * 3, hi=(0.5,) * 3, step_voxels=0.5):
    sc = (ctypes.c_float * 3)()
    of = (ctypes.c_float * 3)()
    st = ctypes.c_float()
    lo_ = (ctypes.c_double * 3)(*lo)
    hi_ = (ctypes.c_double * 3)(*hi)
    _check(lib().plx_grid_geometry(ctypes.cast(_i3(reso), _P), ctypes.cast(lo_, _P),
                                   ctypes.cast(hi_, _P), float(step_voxels), ctypes.cast(sc, _P),
                                   ctypes.cast(of, _P), ctypes.byref(st)))
    return tuple(sc), tuple(of), st.value


def plx_lr_schedule(step, lr0, lr1, max_steps, delay_steps=0.0, delay_mult=1.0) -> float:
    return float(lib().plx_lr_schedule(float(step), float(lr0), float(lr1), float(max_steps),
                                       float(delay_steps), float(delay_mult)))


# --------------------------------------------------------------------- grid

def plx_grid_workspace_bytes(reso) -> int:
    return int(lib().plx_grid_workspace_bytes(ctypes.cast(_i3(reso), _P)))


def plx_mask_count(mask: torch.Tensor, ws=None) -> int:
    out = ctypes.c_int64()
    wp, wb, _keep = _ws(ws, COUNT_WORKSPACE_BYTES, mask.device)
    _check(lib().plx_mask_count(_dptr(mask, "mask", torch.uint8), mask.numel(), wp, wb,
                                ctypes.byref(out), _stream()))
    return int(out.value)


def plx_grid_create(mask: torch.Tensor, reso, index_out: torch.Tensor, ws=None):
    n = int(reso[0]) * int(reso[1]) * int(reso[2])
    wp, wb, _keep = _ws(ws, plx_grid_workspace_bytes(reso), mask.device)
    _check(lib().plx_grid_create(_dptr(mask, "mask", torch.uint8, n), ctypes.cast(_i3(reso), _P),
                                 _dptr(index_out, "index_out", torch.int32, n), wp, wb, _stream()))


def plx_records_pack(sh_dtype, n, density, sh, sigma0, dc, out):
    _check(lib().plx_records_pack(sh_dtype, int(n), _dptr(density, "density", torch.float32),
                                  _dptr(sh, "sh", torch.float32), float(sigma0), float(dc),
                                  _dptr(out, "out"), _stream()))


def plx_records_unpack(sh_dtype, n, records, density=None, sh=None):
    _check(lib().plx_records_unpack(sh_dtype, int(n), _dptr(records, "records"),
                                    _dptr(density, "density", torch.float32),
                                    _dptr(sh, "sh", torch.float32), _stream()))


def plx_records_convert(src_dtype, src, dst_dtype, dst, n):
    _check(lib().plx_records_convert(src_dtype, _dptr(src, "src"), dst_dtype, _dptr(dst, "dst"),
                                     int(n), _stream()))


def plx_grid_build_occupancy(g: PlxGrid, occ_out: torch.Tensor):
    _check(lib().plx_grid_build_occupancy(ctypes.byref(g), _dptr(occ_out, "occ_out", torch.int32),
                                          _stream()))


def plx_grid_prune_count(g: PlxGrid, sigma_thresh, keep_out: torch.Tensor, ws=None):
    kept, pruned = ctypes.c_int64(), ctypes.c_int64()
    wp, wb, _keep = _ws(ws, plx_grid_workspace_bytes(tuple(g.reso)), keep_out.device)
    _check(lib().plx_grid_prune_count(ctypes.byref(g), float(sigma_thresh),
                                      _dptr(keep_out, "keep_out", torch.uint8), wp, wb,
                                      ctypes.byref(kept), ctypes.byref(pruned), _stream()))
    return int(kept.value), int(pruned.value)


def plx_grid_prune_weight_count(g: PlxGrid, wmax: torch.Tensor, w_thresh, keep_out: torch.Tensor,
                                ws=None):
    kept, pruned = ctypes.c_int64(), ctypes.c_int64()
    wp, wb, _keep = _ws(ws, plx_grid_workspace_bytes(tuple(g.reso)), keep_out.device)
    _check(lib().plx_grid_prune_weight_count(ctypes.byref(g), _dptr(wmax, "wmax", torch.float32, g.n_vox),
                                             float(w_thresh),
                                             _dptr(keep_out, "keep_out", torch.uint8), wp, wb,
                                             ctypes.byref(kept), ctypes.byref(pruned), _stream()))
    return int(kept.value), int(pruned.value)


def plx_grid_prune_apply(g: PlxGrid, keep: torch.Tensor, out: PlxGrid, ws=None):
    wp, wb, _keep = _ws(ws, plx_grid_workspace_bytes(tuple(g.reso)), keep.device)
    _check(lib().plx_grid_prune_apply(ctypes.byref(g), _dptr(keep, "keep", torch.uint8),
                                      ctypes.byref(out), wp, wb, _stream()))


def plx_grid_upsample_count(g: PlxGrid, new_reso, ws=None) -> int:
    n = ctypes.c_int64()
    wp, wb, _keep = _ws(ws, COUNT_WORKSPACE_BYTES)
    _check(lib().plx_grid_upsample_count(ctypes.byref(g), ctypes.cast(_i3(new_reso), _P), wp, wb,
                                         ctypes.byref(n), _stream()))
    return int(n.value)


def plx_grid_upsample_apply(g: PlxGrid, out: PlxGrid, ws=None):
    wp, wb, _keep = _ws(ws, plx_grid_workspace_bytes(tuple(out.reso)))
    _check(lib().plx_grid_upsample_apply(ctypes.byref(g), ctypes.byref(out), wp, wb, _stream()))


# --------------------------------------------------------------------- render

def event_handles(events):
    """A C array of the raw HIP handles of 4 torch.cuda.Event objects, for
    plx_render_opts.kernel_events (each event is created by recording it
    once on the current stream; the library records it again)."""
    if events is None:
        return None
    if len(events) != 4:
        raise ValueError("kernel_events takes 4 events")
    for e in events:
        e.record()
    return (ctypes.c_void_p * 4)(*[e.cuda_event for e in events])


def _opts(bg, priors: Priors | None = None, n: int | None = None, grad_bg=None, events=None):
    """bg: one colour (3 numbers) or a device float32 tensor [R, 3] of
    per-ray background colours; priors: the optional priors; grad_bg: device
    float32 [R, 3] that gradient calls fill with dL/d(background colour);
    events: 4 torch.cuda.Event recorded between the render kernels."""
    if isinstance(bg, torch.Tensor):
        o = PlxRenderOpts((ctypes.c_float * 3)(0.0, 0.0, 0.0))
        o.background_rgb = _dptr(bg, "background_rgb", torch.float32, None if n is None else 3 * n)
    else:
        o = PlxRenderOpts((ctypes.c_float * 3)(*[float(x) for x in bg]))
    if grad_bg is not None:
        o.grad_background = _dptr(grad_bg, "grad_bg", torch.float32, None if n is None else 3 * n)
    if priors is not None:
        o.lambda_sparsity = float(priors.lambda_sparsity)
        o.lambda_beta = float(priors.lambda_beta)
        o.beta_eps = float(priors.beta_eps)
        o.reg_loss_sum = _dptr(priors.loss, "priors.loss", torch.float64, 2)
    if events is not None:
        o._events = event_handles(events)  # kept alive with the struct
        o.kernel_events = ctypes.cast(o._events, ctypes.c_void_p)
    return o


def plx_rays_to_ndc(rays_o, rays_d, width, height, focal, near, o_out, d_out):
    n = rays_o.shape[0]
    _check(lib().plx_rays_to_ndc(_dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                 _dptr(rays_d, "rays_d", torch.float32, 3 * n), n, int(width), int(height),
                                 float(focal), float(near), _dptr(o_out, "o_out", torch.float32, 3 * n),
                                 _dptr(d_out, "d_out", torch.float32, 3 * n), _stream()))


def plx_bg_render_fwd(g: PlxGrid, rays_o, rays_d, rgb_out, t_out=None, bg=(1.0, 1.0, 1.0)):
    n = rays_o.shape[0]
    b = (ctypes.c_float * 3)(*[float(x) for x in bg])
    _check(lib().plx_bg_render_fwd(ctypes.byref(g), _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                   _dptr(rays_d, "rays_d", torch.float32, 3 * n), n, b,
                                   _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                   _dptr(t_out, "t_out", torch.float32, n), _stream()))


def plx_bg_render_bwd(g: PlxGrid, rays_o, rays_d, grad_rgb, grad, touched, bg=(1.0, 1.0, 1.0)):
    n = rays_o.shape[0]
    b = (ctypes.c_float * 3)(*[float(x) for x in bg])
    _check(lib().plx_bg_render_bwd(ctypes.byref(g), _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                   _dptr(rays_d, "rays_d", torch.float32, 3 * n), n, b,
                                   _dptr(grad_rgb, "grad_rgb", torch.float32, 3 * n),
                                   _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                   _dptr(touched, "touched", torch.uint8), _stream()))


class Bins:
    """Caller-owned segment lists of one ray batch (plx_bins): the device
    buffers and their descriptor.  Made by make_bins (count, then apply);
    serves every render call on the same rays until the grid's occupancy is
    rebuilt."""

    def __init__(self, desc: PlxBins, ray_buf: torch.Tensor, seg_buf: torch.Tensor | None,
                 samp_buf: torch.Tensor | None = None):
        self.ray_buf, self.seg_buf, self.samp_buf = ray_buf, seg_buf, samp_buf
        self.desc = desc
        desc.ray_buf, desc.ray_buf_bytes = ray_buf.data_ptr(), ray_buf.numel()
        has_seg = seg_buf is not None and seg_buf.numel() > 0
        desc.seg_buf = seg_buf.data_ptr() if has_seg else None
        desc.seg_buf_bytes = seg_buf.numel() if has_seg else 0
        has_samp = samp_buf is not None and samp_buf.numel() > 0
        desc.samp_buf = samp_buf.data_ptr() if has_samp else None
        desc.samp_buf_bytes = samp_buf.numel() if has_samp else 0

    @property
    def n_rays(self) -> int:
        return int(self.desc.n_rays)

    @property
    def n_seg(self) -> int:
        return int(self.desc.n_seg)

    @property
    def n_samp(self) -> int:
        return int(self.desc.n_samp)

    @property
    def n_brick(self) -> int:
        return int(self.desc.n_brick)

    def buffers(self):
        return [self.ray_buf, self.seg_buf, self.samp_buf]


def plx_bins_ray_bytes(reso, n_rays: int) -> int:
    return int(lib().plx_bins_ray_bytes(ctypes.cast(_i3(reso), _P), int(n_rays)))


def plx_bins_seg_bytes(n_seg: int) -> int:
    return int(lib().plx_bins_seg_bytes(int(n_seg)))


def plx_bins_samp_bytes(n_seg: int, n_samp: int) -> int:
    return int(lib().plx_bins_samp_bytes(int(n_seg), int(n_samp)))


def plx_bins_count(g: PlxGrid, rays_o, rays_d, ray_buf: torch.Tensor) -> PlxBins:
    """Phase 1: the descriptor with the rays, the ray buffer and the counts."""
    n = rays_o.shape[0]
    out = PlxBins()
    _check(lib().plx_bins_count(ctypes.byref(g), _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                _dptr(ray_buf, "ray_buf", torch.uint8), ray_buf.numel(),
                                ctypes.byref(out), _stream()))
    return out


def plx_bins_apply(g: PlxGrid, rays_o, rays_d, bins: Bins):
    n = rays_o.shape[0]
    _check(lib().plx_bins_apply(ctypes.byref(g), _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                _dptr(rays_d, "rays_d", torch.float32, 3 * n),
                                ctypes.byref(bins.desc), _stream()))


def plx_bins_verify(g: PlxGrid, bins: Bins):
    _check(lib().plx_bins_verify(ctypes.byref(g), ctypes.byref(bins.desc), _stream()))


def make_bins(g: PlxGrid, rays_o, rays_d, ray_buf: torch.Tensor | None = None,
              seg_buf: torch.Tensor | None = None, samp_buf: torch.Tensor | None = None,
              samples: bool = True) -> Bins:
    """Segment lists of a ray batch: plx_bins_count then plx_bins_apply on
    the current stream, into the given buffers when they are large enough,
    else into new ones.  samples: attach a sample buffer (the recorded
    backward); without one the backward replay scatters its gradients
    itself.  New segment and sample buffers get 1/8 more than this batch
    needs, so that a training loop passing them back in does not allocate
    again for every batch that holds a few more segments than the last."""
    n = rays_o.shape[0]
    need = plx_bins_ray_bytes(tuple(g.reso), n)
    if ray_buf is None or ray_buf.numel() < need:
        ray_buf = workspace(need, rays_o.device)
    desc = plx_bins_count(g, rays_o, rays_d, ray_buf)
    n_seg = int(desc.n_seg)
    if n_seg > 0:
        sneed = plx_bins_seg_bytes(n_seg)
        if seg_buf is None or seg_buf.numel() < sneed:
            seg_buf = workspace(sneed + sneed // 8, rays_o.device)
        if samples:
            pneed = plx_bins_samp_bytes(n_seg, int(desc.n_samp))
            if samp_buf is None or samp_buf.numel() < pneed:
                samp_buf = workspace(pneed + pneed // 8, rays_o.device)
    bins = Bins(desc, ray_buf, seg_buf if n_seg > 0 else None,
                samp_buf if n_seg > 0 and samples else None)
    plx_bins_apply(g, rays_o, rays_d, bins)
    return bins


def _bins_for(g: PlxGrid, rays_o, rays_d, bins: Bins | None) -> Bins:
    return make_bins(g, rays_o, rays_d) if bins is None else bins


# Occupied samples of a ray that the ray-order passes keep at most (20 bytes
# each); a ray with more has the rest evaluated again.
RAY_CAP = 512
# Bytes of a batch's kept samples.  render() holds them until its backward, a
# trainer two sets: at 512 a ray 300,000 rays take 3.1 GB, some eight times
# their segment lists.  Evaluating a sample again costs little: forward and
# backward with 512, 64, 22 and 1 samples kept per ray take 2392, 2430, 2450
# and 2441 us for 300,000 rays (BF16, 512^3 at 5%), 554, 566, 569 and 571 for 65,537
# (FP16, 256^3 at 10%), 288, 313, 327 and 330 for 16,000 (FP32, 512^3), which
# still keep 419.
RAY_SAMP_BYTES = 128 << 20


def ray_cap(n_rays: int, g: PlxGrid | None = None) -> int:
    """Samples kept per ray of a batch: RAY_CAP, or as many as RAY_SAMP_BYTES
    holds, or as a ray of unit direction has on the grid's diagonal."""
    cap = min(RAY_CAP, RAY_SAMP_BYTES // (20 * max(n_rays, 1)))
    # (a grid that the call will refuse has no diagonal)
    if g is not None:
        (nx, ny, nz), (sx, sy, sz), step = g.reso[:], g.scale[:], g.step
        if min(sx, sy, sz, step) > 0:
            steps = math.hypot((nx - 1) / sx, (ny - 1) / sy, (nz - 1) / sz) / step
            if steps < cap:
                cap = int(steps) + 2
    return max(1, cap)


def ray_order(g: PlxGrid, n_rays: int) -> bool:
    """Whether a fused training batch of n_rays rays is run in ray order
    (plx_render_train_rays) rather than over segment lists.  In ray order
    every ray sends a line of atomics per voxel it crosses, and nothing is
    binned, counted or read back; the lists merge the rays of a brick.  The
    batch's occupied brick crossings are estimated by n_rays times the bricks
    along a ray times the share of occupied voxels; the line is 196,608.

    Below it ray order takes at most half the time.  Ray order / lists with
    their binning (us, FP32; crossings): 5000 rays on 256^3 at 10% (48,000) 129 /
    529, on a dense 64^3 (120,000) 127 / 503, 2500 inside a dense 128^3 (120,000)
    286 / 615, 20,000 on 512^3 at 5% (192,000) 317 / 682, 1000 through a dense
    256x256x128 (80,000) 129 / 457.

    Above it ray order is still ahead, up to the recorded backward of 65,536
    rays (5000 inside the 128^3 532 / 822, 20,000 through the 256x256x128 1661 / 2079,
    40,000 on 512^3 495 / 791; 80,000 there 837 / 1484, but 713 / 708 on 256^3 at
    10% and 6481 / 3446 through the 256x256x128).  The lists stay there because
    ray order adds a sample's terms in another order, which a gain below 2 was
    not held to be worth: where a density lies at 0 the last bit of one step
    decides a gate of the next, and with many samples one may.  Two steps of
    20,011 rays through the 256x256x128 grid gave densities that differ by 1e-3
    of the largest in one of eight seeds (else by 1e-6), of 5000 inside the
    128^3 by 4e-6, below the line (64^3, 256^3) by 4e-7; runs of the same order
    differ by 2e-7.  Ray order is not the less exact of the two (densities after a
    step against 64 bits, relative: 6.8e-8 and 7.6e-8 through the 256x256x128,
    3.5e-8 and 4.0e-8 inside the 128^3, 8.8e-8 and 9.8e-8 on 64^3)."""
    b = [-(-(int(r) - 1) // 8) for r in g.reso]
    cells = int(g.reso[0]) * int(g.reso[1]) * int(g.reso[2])
    return n_rays * sum(b) * int(g.n_vox) < 3 * 65536 * cells


def ray_order_grad(g: PlxGrid, n_rays: int) -> bool:
    """As ray_order, for a separate forward and backward pass, where lists
    also cost a forward of their own and no step follows: ray order while few
    rays cross a brick (x = n_rays times the bricks along a ray over all
    bricks), and for small batches, whose lists are mostly fixed costs.  Ray
    order / lists in us: 5000 rays on 64^3 132 / 214; sparse grids (up to a
    quarter occupied): 300,000 on 512^3 at 5% (x = 73) 2442 / 3762 (BF16), 400,000
    (98) 3184 / 3174, 230,400 on 380^3 at 10% (100) 2852 / 2873, 300,000 (130) 3635 /
    3190, 100,000 on 256^3 at 10% (98) 801 / 858 (FP16), 64,000 on 128^3 at 12%
    (250) 384 / 442; dense grids: 128^3 from outside (47) 505 / 759, from inside (31)
    804 / 906, but 16,384 there (64) 1551 / 1370; 20,000 through a 256x256x128 (33)
    1674 / 2442, 49,152 (80) 4092 / 3704."""
    b = [-(-(int(r) - 1) // 8) for r in g.reso]
    sparse = 4 * int(g.n_vox) < int(g.reso[0]) * int(g.reso[1]) * int(g.reso[2])
    return (n_rays < (65536 if sparse else 8192)
            or n_rays * sum(b) < 3 * (100 if sparse else 50) * b[0] * b[1] * b[2])


class RayWork:
    """Scratch of one gradient batch in ray order, taken by plx_render_train
    in place of segment lists."""

    def __init__(self, n_rays: int, ray_ws: torch.Tensor, samp_ws: torch.Tensor, cap: int):
        self.n_rays, self.ray_ws, self.samp_ws, self.cap = n_rays, ray_ws, samp_ws, cap

    def buffers(self):
        """As of Bins, which may take the buffers over and hand them back."""
        return [self.ray_ws, self.samp_ws, None]


def make_ray_work(n_rays: int, ray_ws: torch.Tensor | None = None, samp_ws: torch.Tensor | None = None,
                  device=None, cap: int | None = None) -> RayWork:
    """Scratch for n_rays rays, in the given buffers when they are large
    enough, else in new ones.  cap: samples kept per ray (ray_cap)."""
    if cap is None:
        cap = ray_cap(n_rays)
    need = plx_rays_ray_bytes(n_rays), plx_rays_samp_bytes(n_rays, cap)
    if ray_ws is None or ray_ws.numel() < need[0]:
        ray_ws = workspace(need[0], device)
    if samp_ws is None or samp_ws.numel() < need[1]:
        samp_ws = workspace(need[1], device)
    return RayWork(n_rays, ray_ws, samp_ws, cap)


def plx_render_fwd(g: PlxGrid, rays_o, rays_d, rgb_out, tau_out=None, bg=(1.0, 1.0, 1.0),
                   bins: Bins | None = None, events=None):
    """bins: the batch's segment lists where they exist already.  Without them
    the rays are marched in ray order, which needs none; only very large
    batches of scattered rays on dense 16-bit grids would gain from lists made
    for the purpose (640,000 on 128^3 2.96 ms, over lists with their binning
    2.22; an image of as many pixels 1.53 and 2.66)."""
    n = rays_o.shape[0]
    o = _opts(bg, None, n, None, events)
    if bins is None:
        plx_render_fwd_rays(g, rays_o, rays_d, rgb_out, tau_out, None, bg, events)
        return
    b = bins
    _check(lib().plx_render_fwd(ctypes.byref(g), ctypes.byref(o),
                                _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                ctypes.byref(b.desc),
                                _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                _dptr(tau_out, "tau_out", torch.float32, n), _stream()))


def plx_render_bwd(g: PlxGrid, rays_o, rays_d, grad_rgb, tau_fwd, grad, touched,
                   bg=(1.0, 1.0, 1.0), priors: Priors | None = None, grad_bg=None,
                   bins: Bins | None = None, events=None):
    n = rays_o.shape[0]
    o = _opts(bg, priors, n, grad_bg, events)
    b = _bins_for(g, rays_o, rays_d, bins)
    _check(lib().plx_render_bwd(ctypes.byref(g), ctypes.byref(o),
                                _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                ctypes.byref(b.desc),
                                _dptr(grad_rgb, "grad_rgb", torch.float32, 3 * n),
                                _dptr(tau_fwd, "tau_fwd", torch.float32, n),
                                _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                _dptr(touched, "touched", torch.uint8), _stream()))


def plx_render_train(g: PlxGrid, rays_o, rays_d, target, loss_scale, grad, touched, loss_sum,
                     rgb_out=None, bg=(1.0, 1.0, 1.0), priors: Priors | None = None, grad_bg=None,
                     bins: Bins | RayWork | None = None, events=None):
    """bins: the batch's segment lists, or scratch for a batch in ray order;
    made here (by ray_order) when not given."""
    n = rays_o.shape[0]
    if bins is None and ray_order(g, n):
        bins = make_ray_work(n, device=rays_o.device, cap=ray_cap(n, g))
    if isinstance(bins, RayWork):
        plx_render_train_rays(g, rays_o, rays_d, target, loss_scale, grad, touched, loss_sum, bins, rgb_out, bg,
                              priors, grad_bg, events)
        return
    o = _opts(bg, priors, n, grad_bg, events)
    b = _bins_for(g, rays_o, rays_d, bins)
    _check(lib().plx_render_train(ctypes.byref(g), ctypes.byref(o),
                                  _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                  _dptr(rays_d, "rays_d", torch.float32, 3 * n),
                                  _dptr(target, "target", torch.float32, 3 * n), n,
                                  ctypes.byref(b.desc), float(loss_scale), _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                  _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                  _dptr(touched, "touched", torch.uint8),
                                  _dptr(loss_sum, "loss_sum", torch.float64, 1), _stream()))


def plx_render_train_static(g: PlxGrid, rays_o, rays_d, target, loss_scale, grad, touched, loss_sum,
                            rgb_out=None, bg=(1.0, 1.0, 1.0), priors: Priors | None = None,
                            grad_bg=None, events=None):
    """plx_render_train with the segment lists in the library's fixed
    scratch: allocates nothing and never synchronises (PlxError with code
    PLX_ENOMEM when the batch does not fit the scratch)."""
    n = rays_o.shape[0]
    o = _opts(bg, priors, n, grad_bg, events)
    _check(lib().plx_render_train_static(ctypes.byref(g), ctypes.byref(o),
                                         _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                         _dptr(rays_d, "rays_d", torch.float32, 3 * n),
                                         _dptr(target, "target", torch.float32, 3 * n), n,
                                         float(loss_scale), _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                         _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                         _dptr(touched, "touched", torch.uint8),
                                         _dptr(loss_sum, "loss_sum", torch.float64, 1), _stream()))


def plx_rays_ray_bytes(n_rays: int) -> int:
    return int(lib().plx_rays_ray_bytes(int(n_rays)))


def plx_rays_samp_bytes(n_rays: int, cap: int) -> int:
    return int(lib().plx_rays_samp_bytes(int(n_rays), int(cap)))


def _work_args(work: RayWork | None, n: int):
    if work is None:
        return None, 0, None, 0, 0
    if work.n_rays != n:
        raise ValueError(f"scratch made for {work.n_rays} rays, the call has {n}")
    return (_dptr(work.ray_ws, "ray_ws", torch.uint8), work.ray_ws.numel(), _dptr(work.samp_ws, "samp_ws", torch.uint8),
            work.samp_ws.numel(), int(work.cap))


def plx_render_fwd_rays(g: PlxGrid, rays_o, rays_d, rgb_out, tau_out=None, work: RayWork | None = None,
                        bg=(1.0, 1.0, 1.0), events=None):
    """plx_render_fwd in ray order; with work (make_ray_work) the occupied
    samples are kept there for plx_render_bwd_rays."""
    n = rays_o.shape[0]
    o = _opts(bg, None, n, None, events)
    _check(lib().plx_render_fwd_rays(ctypes.byref(g), ctypes.byref(o),
                                     _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                     _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                     _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                     _dptr(tau_out, "tau_out", torch.float32, n), *_work_args(work, n), _stream()))


def plx_render_bwd_rays(g: PlxGrid, rays_o, rays_d, grad_rgb, work: RayWork, grad, touched, bg=(1.0, 1.0, 1.0),
                        priors: Priors | None = None, grad_bg=None, events=None):
    n = rays_o.shape[0]
    o = _opts(bg, priors, n, grad_bg, events)
    _check(lib().plx_render_bwd_rays(ctypes.byref(g), ctypes.byref(o),
                                     _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                     _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                     _dptr(grad_rgb, "grad_rgb", torch.float32, 3 * n), *_work_args(work, n),
                                     _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                     _dptr(touched, "touched", torch.uint8), _stream()))


def plx_render_train_rays(g: PlxGrid, rays_o, rays_d, target, loss_scale, grad, touched, loss_sum, work: RayWork,
                          rgb_out=None, bg=(1.0, 1.0, 1.0), priors: Priors | None = None, grad_bg=None,
                          events=None):
    """plx_render_train in ray order, with work (make_ray_work) as scratch."""
    n = rays_o.shape[0]
    o = _opts(bg, priors, n, grad_bg, events)
    _check(lib().plx_render_train_rays(ctypes.byref(g), ctypes.byref(o),
                                       _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                       _dptr(rays_d, "rays_d", torch.float32, 3 * n),
                                       _dptr(target, "target", torch.float32, 3 * n), n, *_work_args(work, n),
                                       float(loss_scale), _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                       _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                       _dptr(touched, "touched", torch.uint8),
                                       _dptr(loss_sum, "loss_sum", torch.float64, 1), _stream()))


def plx_render_state_bytes(n_rays: int, cap: int) -> int:
    return int(lib().plx_render_state_bytes(int(n_rays), int(cap)))


def _state_ptr(state, n, cap):
    need = plx_render_state_bytes(n, cap)
    if not (isinstance(state, torch.Tensor) and state.is_cuda and state.dtype == torch.uint8
            and state.is_contiguous() and state.numel() >= need):
        raise ValueError(f"state must be a contiguous CUDA uint8 tensor of >= {need} bytes")
    return ctypes.c_void_p(state.data_ptr()), state.numel()


def plx_render_max_weight(g: PlxGrid, rays_o, rays_d, wmax, bins: Bins | None = None):
    n = rays_o.shape[0]
    b = make_bins(g, rays_o, rays_d, samples=False) if bins is None else bins
    _check(lib().plx_render_max_weight(ctypes.byref(g),
                                       _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                       _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                       ctypes.byref(b.desc),
                                       _dptr(wmax, "wmax", torch.float32, g.n_vox), _stream()))


def plx_render_fwd_state(g: PlxGrid, rays_o, rays_d, rgb_out, tau_out, state, cap,
                         bg=(1.0, 1.0, 1.0)):
    n = rays_o.shape[0]
    o = _opts(bg, None, n)
    sp, sb = _state_ptr(state, n, cap)
    _check(lib().plx_render_fwd_state(ctypes.byref(g), ctypes.byref(o),
                                      _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                      _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                      _dptr(rgb_out, "rgb_out", torch.float32, 3 * n),
                                      _dptr(tau_out, "tau_out", torch.float32, n), sp, sb, int(cap),
                                      _stream()))


def plx_render_bwd_state(g: PlxGrid, rays_o, rays_d, grad_rgb, tau_fwd, state, cap, grad, touched,
                         bg=(1.0, 1.0, 1.0), priors: Priors | None = None, grad_bg=None):
    n = rays_o.shape[0]
    o = _opts(bg, priors, n, grad_bg)
    sp, sb = _state_ptr(state, n, cap)
    _check(lib().plx_render_bwd_state(ctypes.byref(g), ctypes.byref(o),
                                      _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                      _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                      _dptr(grad_rgb, "grad_rgb", torch.float32, 3 * n),
                                      _dptr(tau_fwd, "tau_fwd", torch.float32, n), sp, sb, int(cap),
                                      _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                      _dptr(touched, "touched", torch.uint8), _stream()))


class SceneTable:
    """Device copy of the descriptors of resident scenes (plx_scene_table_set),
    the scene argument of plx_render_views.  Keeps the grids referenced."""

    def __init__(self, scenes, stream=None):
        self.grids = list(scenes)
        descs = [g.desc() for g in self.grids]
        if not descs:
            raise ValueError("need at least one scene")
        self.n_scenes = len(descs)
        self.sh_dtype = int(descs[0].sh_dtype)
        self.buf = workspace(plx_scene_table_bytes(self.n_scenes), self.grids[0].device)
        sc = (PlxGrid * self.n_scenes)(*descs)
        s = ctypes.c_void_p((stream or torch.cuda.current_stream()).cuda_stream)
        _check(lib().plx_scene_table_set(ctypes.cast(sc, _GP), self.n_scenes, _dptr(self.buf, "table", torch.uint8),
                                         self.buf.numel(), s))


def plx_scene_table_bytes(n_scenes: int) -> int:
    return int(lib().plx_scene_table_bytes(int(n_scenes)))


VIEWS_QUEUE_BYTES = 256


def views_queue(device=None) -> torch.Tensor:
    """A queue buffer for plx_render_views (zero-filled, as the call needs)."""
    return torch.zeros(VIEWS_QUEUE_BYTES, dtype=torch.uint8, device=device if device is not None else "cuda")


# Views from this many pixels on may take a lane per ray.
LANE_MIN_PIXELS = 1 << 17
VIEW_LANE = 1  # PLX_VIEW_LANE


def view_by_lane(v: PlxView, grid) -> bool:
    """Whether a view of a grid takes a lane per ray (PLX_VIEW_LANE): when the
    rays of a tile lie so close that its lanes read the same few records, each
    lane's corners kept from sample to sample cost less than the march by
    several lanes.  The pixels' pitch at the grid's centre (or at half the
    grid's extent, from inside), in voxels, tells it for every resolution,
    occupancy and distance.  Several lanes / one in ms, FP32: pitch 0.32 2.50 /
    2.62 (256^3 at 25%), 0.25 3.36 / 3.04 (dense 200^3), 0.17 6.46 / 5.55 (dense
    128^3), 0.13 21.7 / 16.9 (512^3 at 5%), 0.03 25.2 / 11.2 (dense 128^3); 16 bits: 0.17
    3.50 / 4.00 (dense 128^3), 0.11 20.0 / 19.8 (256^3 at 25%), 0.08 9.67 / 8.33 (dense
    200^3), 0.03 13.4 / 8.9 (dense 128^3).  A view's colours depend on it and its
    scene alone: the choice does not see the rest of the list."""
    if v.width * v.height < LANE_MIN_PIXELS:
        return False
    n = grid.reso
    x = [v.c2w[4 * a + 3] * float(grid.scale[a]) + float(grid.offset[a]) - 0.5 * (n[a] - 1) for a in range(3)]
    depth = max(math.sqrt(sum(t * t for t in x)), 0.5 * max(n))
    return depth < (0.2 if grid.sh_dtype == PLX_F32 else 0.1) * v.focal


def plx_render_views(table: SceneTable, views, rgb_out, queue, bg=(1.0, 1.0, 1.0), stream=None):
    """table: SceneTable; views: list of PlxView; rgb_out: device float32
    tensor; queue: views_queue().  stream: a torch.cuda.Stream (default: the
    current stream).  Asynchronous."""
    vw = (PlxView * max(len(views), 1))(*views)
    for v in vw[:len(views)]:
        if 0 <= v.scene < table.n_scenes and view_by_lane(v, table.grids[v.scene]):
            v.reserved |= VIEW_LANE
    o = _opts(bg)
    s = ctypes.c_void_p((stream or torch.cuda.current_stream()).cuda_stream)
    _check(lib().plx_render_views(_dptr(table.buf, "table", torch.uint8), table.n_scenes, table.sh_dtype,
                                  ctypes.cast(vw, _P), len(views), ctypes.byref(o),
                                  _dptr(rgb_out, "rgb_out", torch.float32),
                                  _dptr(queue, "queue", torch.uint8, VIEWS_QUEUE_BYTES), s))


def plx_render_views_status(queue, stream=None):
    s = ctypes.c_void_p((stream or torch.cuda.current_stream()).cuda_stream)
    _check(lib().plx_render_views_status(_dptr(queue, "queue", torch.uint8), s))


def plx_render_stats(g: PlxGrid, rays_o, rays_d, cell_mark, vox_mark, ws=None):
    n = rays_o.shape[0]
    counts = (ctypes.c_int64 * 4)()
    wp, wb, _keep = _ws(ws, COUNT_WORKSPACE_BYTES, rays_o.device)
    _check(lib().plx_render_stats(ctypes.byref(g), _dptr(rays_o, "rays_o", torch.float32, 3 * n),
                                  _dptr(rays_d, "rays_d", torch.float32, 3 * n), n,
                                  _dptr(cell_mark, "cell_mark", torch.int32),
                                  _dptr(vox_mark, "vox_mark", torch.int32), wp, wb,
                                  ctypes.cast(counts, _P), _stream()))
    return tuple(int(c) for c in counts)


# --------------------------------------------------------------------- TV / optimiser

def plx_tv_grad(g: PlxGrid, cell_start, cell_count, lambda_sigma, lambda_sh, eps, grad, touched,
                loss_sum=None):
    _check(lib().plx_tv_grad(ctypes.byref(g), int(cell_start), int(cell_count), float(lambda_sigma),
                             float(lambda_sh), float(eps),
                             _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                             _dptr(touched, "touched", torch.uint8),
                             _dptr(loss_sum, "loss_sum", torch.float64, 1), _stream()))


def plx_bg_tv_grad(g: PlxGrid, cell_start, cell_count, lambda_sigma, lambda_color, eps, grad, touched,
                   loss_sum=None):
    _check(lib().plx_bg_tv_grad(ctypes.byref(g), int(cell_start), int(cell_count), float(lambda_sigma),
                                float(lambda_color), float(eps),
                                _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                _dptr(touched, "touched", torch.uint8),
                                _dptr(loss_sum, "loss_sum", torch.float64, 1), _stream()))


def plx_touched_count(touched, n_vox, ws=None) -> int:
    out = ctypes.c_int64()
    wp, wb, _keep = _ws(ws, COUNT_WORKSPACE_BYTES, touched.device)
    _check(lib().plx_touched_count(_dptr(touched, "touched", torch.uint8), int(n_vox), wp, wb,
                                   ctypes.byref(out), _stream()))
    return int(out.value)


def plx_rmsprop_step(g: PlxGrid, master, vstate, grad, touched, lr_sigma, lr_sh, beta=0.95,
                     eps=1e-8):
    _check(lib().plx_rmsprop_step(ctypes.byref(g), _dptr(master, "master", torch.float32),
                                  _dptr(vstate, "vstate", torch.float32, REC_SLOTS * g.n_vox),
                                  _dptr(grad, "grad", torch.float32, REC_SLOTS * g.n_vox),
                                  _dptr(touched, "touched", torch.uint8), float(lr_sigma),
                                  float(lr_sh), float(beta), float(eps), _stream()))
