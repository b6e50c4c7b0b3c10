"""Tensor-level convenience layer over ``binding``: allocates outputs and the
workspace with torch on the tensor's device and enqueues on torch's current
stream.  Plumbing only -- every arithmetic step runs inside libgf.so, and the
steps around it (checks, allocation, stream and workspace look-up) in one native
call per function (``csrc_host/gf_torch.cpp``)."""
from __future__ import annotations

import os

import torch

from . import binding as B
from .workloads import Layer


def desc_for(layer: Layer, N: int, r: int, dtype: str) -> B.ConvDesc:
    return B.ConvDesc(N=N, C_in=layer.C_in, C_out=layer.C_out, H_in=layer.H, W_in=layer.W,
                      K_h=layer.K, K_w=layer.K, stride=layer.stride, pad=layer.pad,
                      dilation=layer.dilation, groups=layer.groups, r=r,
                      dtype=B.GF_BF16 if dtype == "bf16" else B.GF_F32)


def _tdtype(d: B.ConvDesc):
    return torch.bfloat16 if d.dtype == B.GF_BF16 else torch.float32


def _check(t: torch.Tensor, d: B.ConvDesc, shape, what: str, dtype=None):
    if not t.is_cuda or not t.is_contiguous():
        raise ValueError(f"{what} must be a contiguous device tensor")
    if tuple(t.shape) != tuple(shape):
        raise ValueError(f"{what}: expected shape {tuple(shape)}, got {tuple(t.shape)}")
    if t.dtype != (dtype or _tdtype(d)):
        raise ValueError(f"{what}: expected dtype {dtype or _tdtype(d)}, got {t.dtype}")


def shapes(d: B.ConvDesc) -> dict:
    Hy, Wy, Hp, Wp = B.gf_out_shape(d)
    cg = d.C_in // d.groups
    return {
        "x": (d.N, d.C_in, d.H_in, d.W_in), "g_y": (d.N, d.C_out, Hy, Wy),
        "w": (d.C_out, cg, d.K_h, d.K_w),
        "x_u": (d.N, d.C_in, d.H_in, d.W_in) if d.r == 1 else (d.N, d.C_in, Hp, Wp),
        "gy_u": (d.N, d.C_out, Hp, Wp),
        "g_x_u": (d.N, d.C_in, d.H_in, d.W_in) if d.r == 1 else (d.N, d.C_in, Hp, Wp),
    }


class Workspace:
    """A reusable device scratch buffer (grown on demand, never inside a call to libgf).  One
    Workspace serves ONE stream at a time: two calls that may run concurrently need two."""

    def __init__(self, device="cuda"):
        self.device = device
        self.buf = None

    def get(self, nbytes: int):
        if nbytes == 0:
            return 0, 0
        if self.buf is None or self.buf.numel() < nbytes:
            if self.buf is not None:
                # the old buffer goes back to the caching allocator: tell it that work already
                # enqueued on the current stream may still be using it
                self.buf.record_stream(torch.cuda.current_stream(self.buf.device))
            self.buf = torch.empty(max(nbytes, 256), dtype=torch.uint8, device=self.device)
        return int(self.buf.data_ptr()), int(self.buf.numel())


class _Native:
    """The native module, loaded (with libgf.so) by the first call; fails loudly if it was not built."""

    def __getattr__(self, name):
        path = os.path.join(B.HERE, "_gf_torch.so")
        if not os.path.exists(path):
            raise ImportError(f"{path} is missing: build it with `python -m paper_2301_00330_amd.build` (needs hipcc)")
        B.lib()   # libgf.so first: the module links against it
        from . import _gf_torch
        _gf_torch.setup(_check, B.GfError, Workspace, torch.int8, torch.OutOfMemoryError)
        self.__dict__.update((k, v) for k, v in vars(_gf_torch).items() if not k.startswith("_"))
        return self.__dict__[name]


_C = _Native()

# Every function below takes ``ws``, the caller's workspace; None: a default one per (device, current stream),
# since calls on different streams may overlap in time and must not share scratch memory.


def pool_activation(d: B.ConvDesc, x: torch.Tensor, out: torch.Tensor | None = None):
    return _C.pool_activation(d, x, out)


def pool_activation_batch(descs, xs):
    """x_u of several layers from one launch (gf_pool_activation_batch)."""
    return _C.pool_activation_batch(descs, xs)


def pool_activation_batch_q8(descs, xs, inv_deltas):
    """x_q of several layers from one launch (gf_pool_activation_batch_q8)."""
    return _C.pool_activation_batch_q8(descs, xs, inv_deltas)


def pool_activation_mask(d: B.ConvDesc, x: torch.Tensor, hi: float = float("inf")):
    """(x_u, m_u): patch sums of x and the share of each patch with 0 < x < hi (the gradient mask of the
    ReLU / clipped ReLU that produced x, averaged over the patch)."""
    return _C.pool_activation_mask(d, x, hi)


def filter_grad(d: B.ConvDesc, g_y: torch.Tensor, out: torch.Tensor | None = None):
    return _C.filter_grad(d, g_y, out)


def conv_bwd_weight(d: B.ConvDesc, x_u: torch.Tensor, gy_u: torch.Tensor,
                    out: torch.Tensor | None = None, ws: Workspace | None = None):
    return _C.conv_bwd_weight(d, x_u, gy_u, out, ws)


def conv_bwd_input(d: B.ConvDesc, gy_u: torch.Tensor, w: torch.Tensor, reduced_out: bool = False,
                   out: torch.Tensor | None = None, ws: Workspace | None = None):
    return _C.conv_bwd_input(d, gy_u, w, reduced_out, out, ws)


def conv_bwd_filtered(d: B.ConvDesc, g_y: torch.Tensor, x_u: torch.Tensor, w: torch.Tensor,
                      want_gyu: bool = True, ws: Workspace | None = None):
    """(g_w, g_x, gy_u or None) from one call of gf_conv_bwd_filtered."""
    return _C.conv_bwd_filtered(d, g_y, x_u, w, want_gyu, ws)


def filter_grad_snr(d: B.ConvDesc, g_y: torch.Tensor, ws: Workspace | None = None):
    """(gy_u, stats) with stats = [sum g_y^2, sum (g_y - patch mean)^2] as a float64 device tensor."""
    return _C.filter_grad_snr(d, g_y, ws)


def conv_bwd_chained(d: B.ConvDesc, gy_u: torch.Tensor, x_u: torch.Tensor, w: torch.Tensor,
                     reduced_out: bool = True, mask_u: torch.Tensor | None = None, ws: Workspace | None = None):
    """(g_w, g_x) from one call of gf_conv_bwd_chained; g_x is the reduced map unless reduced_out is False.
    mask_u (from pool_activation_mask of this layer's input) is multiplied into the reduced g_x."""
    return _C.conv_bwd_chained(d, gy_u, x_u, w, reduced_out, mask_u, ws)


def conv_bwd_exact(d: B.ConvDesc, x, w, g_y, want_gw: bool = True, want_gx: bool = True,
                   ws: Workspace | None = None):
    return _C.conv_bwd_exact(d, x, w, g_y, want_gw, want_gx, ws)


# ---- gradient filtering on signed 8-bit codes (one step size per tensor, chosen by the caller) ----

def filter_grad_q8(d: B.ConvDesc, g_y: torch.Tensor, inv_delta: float) -> torch.Tensor:
    return _C.filter_grad_q8(d, g_y, inv_delta)


def pool_activation_q8(d: B.ConvDesc, x: torch.Tensor, inv_delta: float) -> torch.Tensor:
    return _C.pool_activation_q8(d, x, inv_delta)


def kernel_sum_q8(d: B.ConvDesc, w: torch.Tensor, inv_delta: float) -> torch.Tensor:
    return _C.kernel_sum_q8(d, w, inv_delta)


def conv_bwd_unique(d: B.ConvDesc, gy_u: torch.Tensor, x_u: torch.Tensor, w: torch.Tensor, reduced_out: bool = False,
                    ws: Workspace | None = None):
    """(g_w, g_x) of gf_conv_bwd_unique: vanilla BP of the layer's kernel on the patch grid."""
    return _C.conv_bwd_unique(d, gy_u, x_u, w, reduced_out, ws)


def conv_bwd_weight_q8(d: B.ConvDesc, x_q: torch.Tensor, gy_q: torch.Tensor, scale: float,
                       ws: Workspace | None = None) -> torch.Tensor:
    return _C.conv_bwd_weight_q8(d, x_q, gy_q, scale, ws)


def conv_bwd_filtered_q8(d: B.ConvDesc, g_y: torch.Tensor, inv_delta_gy: float, x_q: torch.Tensor, w: torch.Tensor,
                         inv_delta_w: float, scale_w: float, scale_x: float, want_gyq: bool = False,
                         ws: Workspace | None = None):
    """Filter with code output + kernel-sum codes + Eq. 5 and Eq. 3 on codes in one call: (g_w, g_x[, gy_q])."""
    return _C.conv_bwd_filtered_q8(d, g_y, inv_delta_gy, x_q, w, inv_delta_w, scale_w, scale_x, want_gyq, ws)


def conv_bwd_input_q8(d: B.ConvDesc, gy_q: torch.Tensor, w_q: torch.Tensor, scale: float,
                      reduced_out: bool = False, ws: Workspace | None = None) -> torch.Tensor:
    return _C.conv_bwd_input_q8(d, gy_q, w_q, scale, reduced_out, ws)
