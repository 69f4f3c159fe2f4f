"""Thin ctypes binding of the group-layer-normalization entry points of libmtfm_hta.so (C ABI declared in
include/mtfm_gln.h).  Argument marshalling only; PyTorch supplies device memory and the stream.  There is no
fallback: without the built library the first call raises."""
from __future__ import annotations

import ctypes
import struct
from typing import Optional, Tuple

import torch

from . import hta

EXPORTS = ("mtfm_gln_fwd", "mtfm_gln_bwd", "mtfm_gln_bwd_workspace_bytes", "mtfm_gln_validate_host")
KERNEL_FWD, KERNEL_BWD, KERNEL_BWD_REDUCE = 4, 5, 6

_declared = False

# argument block of mtfm_binding_gln (struct GlnArgs of csrc/binding.hip), see hta.call_packed
_BLOCK = struct.Struct("14P3q2ifi")


def load_library() -> ctypes.CDLL:
    global _declared
    lib = hta.load_library()
    if not _declared:
        vp, i32, i64, f32, sz, ci = (ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_float, ctypes.c_size_t,
                                     ctypes.c_int)
        lib.mtfm_gln_fwd.restype = ci
        lib.mtfm_gln_fwd.argtypes = [vp] * 8 + [i64, i32, i32, f32, ci, vp]
        lib.mtfm_gln_bwd_workspace_bytes.restype = sz
        lib.mtfm_gln_bwd_workspace_bytes.argtypes = [i32, i32]
        lib.mtfm_gln_bwd.restype = ci
        lib.mtfm_gln_bwd.argtypes = [vp] * 12 + [i64, i32, i32, ci, vp, sz, vp]
        lib.mtfm_gln_validate_host.restype = ci
        lib.mtfm_gln_validate_host.argtypes = [vp, i64, i32]
        _declared = True
    return lib


def _dtype_code(t: torch.Tensor) -> int:
    if t.dtype == torch.bfloat16:
        return hta.BF16
    if t.dtype == torch.float32:
        return hta.FP32
    raise TypeError(f"unsupported element type {t.dtype}")


def _check(status: int) -> None:
    if status != hta.OK:
        raise hta.HtaError(status, hta.mtfm_hta_last_error())


def _ptr(t: Optional[torch.Tensor]) -> int:
    return 0 if t is None else t.data_ptr()


def mtfm_gln_bwd_workspace_bytes(d_model: int, n_groups: int) -> int:
    return int(load_library().mtfm_gln_bwd_workspace_bytes(d_model, n_groups))


def mtfm_gln_validate_host(group_id: torch.Tensor, n_groups: int) -> None:
    g = group_id.detach().to("cpu", torch.int32).contiguous()
    _check(load_library().mtfm_gln_validate_host(g.data_ptr(), g.numel(), n_groups))


def mtfm_gln_fwd(x: torch.Tensor, group_id: torch.Tensor, gamma: torch.Tensor, beta: torch.Tensor, eps: float,
                 gate: Optional[torch.Tensor] = None, y: Optional[torch.Tensor] = None,
                 save_stats: bool = True, stats=None) -> Tuple[torch.Tensor, Optional[torch.Tensor], Optional[torch.Tensor]]:
    """y = GLN(x) (times gate); returns (y, mean, rstd), the statistics being None when save_stats is False.
    `stats` may hold preallocated (mean, rstd) tensors."""
    lib = load_library()
    n, d = x.shape
    if y is None:
        y = torch.empty_like(x)
    if stats is not None:
        mean, rstd = stats
    elif save_stats:
        mean = torch.empty(n, dtype=torch.float32, device=x.device)
        rstd = torch.empty(n, dtype=torch.float32, device=x.device)
    else:
        mean = rstd = None
    status = lib.mtfm_binding_gln(_BLOCK.pack(
        x.data_ptr(), _ptr(gate), group_id.data_ptr(), gamma.data_ptr(), beta.data_ptr(), y.data_ptr(), _ptr(mean),
        _ptr(rstd), 0, 0, 0, 0, 0, 0, 0, n, 0, d, gamma.shape[0], eps, _dtype_code(x)), hta._current_stream())
    if status != hta.OK:
        _check(status)
    return y, mean, rstd


def mtfm_gln_bwd(dy: torch.Tensor, x: torch.Tensor, group_id: torch.Tensor, gamma: torch.Tensor,
                 beta: Optional[torch.Tensor], mean: torch.Tensor, rstd: torch.Tensor,
                 gate: Optional[torch.Tensor] = None, workspace: Optional[torch.Tensor] = None, out=None):
    """Returns (dx, dgamma, dbeta, dgate); dgate is None without a gate.  `out` may hold preallocated
    (dx, dgamma, dbeta, dgate) tensors."""
    lib = load_library()
    n, d = x.shape
    groups = gamma.shape[0]
    if out is None:
        out = (torch.empty_like(x), torch.empty_like(gamma), torch.empty_like(gamma),
               None if gate is None else torch.empty_like(x))
    dx, dgamma, dbeta, dgate = out
    if workspace is None:
        workspace = torch.empty(max(mtfm_gln_bwd_workspace_bytes(d, groups), 256), dtype=torch.uint8, device=x.device)
    status = lib.mtfm_binding_gln(_BLOCK.pack(
        x.data_ptr(), _ptr(gate), group_id.data_ptr(), gamma.data_ptr(), _ptr(beta), 0, mean.data_ptr(), rstd.data_ptr(),
        dy.data_ptr(), dx.data_ptr(), _ptr(dgate), dgamma.data_ptr(), dbeta.data_ptr(), workspace.data_ptr(),
        workspace.numel(), n, 1, d, groups, 0.0, _dtype_code(x)), hta._current_stream())
    if status != hta.OK:
        _check(status)
    return dx, dgamma, dbeta, dgate
