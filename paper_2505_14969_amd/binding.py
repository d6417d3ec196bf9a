"""Thin binding of libstree.so: argument marshalling only.

Every function takes torch tensors that already live on the GPU, passes their
device pointers and the current HIP stream through the C ABI declared in
``include/stree.h`` and returns the output tensors.  The checks, the results'
allocation and the marshalling of a call are native code (``csrc/host.cpp``,
``_host.so``).  No step of the path is computed here, and there is no CPU
fallback: if the library is missing ``load()`` raises, and every call on tensors
does if either is.
"""
from __future__ import annotations

import ctypes as C
import os
from typing import Optional, Tuple

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libstree.so")

F32, BF16 = 0, 1
FLAG_CONV_SILU = 1
FLAG_DT_SOFTPLUS = 2
FLAG_FORCE_FMA = 256
FLAG_GENERAL_MFMA = 1024
MAX_NODES = 256


class StreeDims(C.Structure):
    _fields_ = [(n, C.c_int32) for n in ("batch", "nnodes", "nheads", "headdim", "dstate", "ngroups",
                                         "conv_width", "io_dtype", "state_dtype", "flags")] + \
               [(n, C.c_int64) for n in ("x_stride_n", "b_stride_n", "c_stride_n")] + [("dt_bias", C.c_void_p)]


class StreeReplay(C.Structure):
    _fields_ = [("nnodes", C.c_int32), ("reserved", C.c_int32), ("parent", C.c_void_p), ("accepted", C.c_void_p),
                ("x", C.c_void_p), ("dt", C.c_void_p), ("Bm", C.c_void_p),
                ("x_stride_n", C.c_int64), ("b_stride_n", C.c_int64)]


class StreeError(RuntimeError):
    def __init__(self, code: int, where: str):
        self.code = code
        msg = load().stree_status_string(code).decode()
        super().__init__(f"{where}: status {code} ({msg})")


_lib = None
_host = None           # the native module, bound to the library's entry points
_VP = C.c_void_p
_ENTRIES = ("tree_conv", "tree_ssd", "commit_state", "tree_ssd_replay", "tree_conv_replay", "tree_step", "gate_norm",
            "linear_ssd")


def _bind(lib: C.CDLL) -> None:
    """Point the native module at the entry points of `lib`."""
    global _host
    try:
        from . import _host as host
    except ImportError as e:
        raise ImportError(f"{os.path.join(_HERE, '_host.so')} is not built for this torch; run "
                          "paper_2505_14969_amd/build.py") from e
    host.bind(StreeError, *(C.cast(getattr(lib, "stree_" + n), _VP).value for n in _ENTRIES))
    _host = host


def _native():
    if _host is None:
        _bind(load())
    return _host


def load() -> C.CDLL:
    """Load libstree.so (build it first with ``python -m paper_2505_14969_amd.build``
    or ``__graft_entry__.build()``).  Raises if it is not there."""
    global _lib, _host
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise FileNotFoundError(f"{LIB_PATH} is not built; run paper_2505_14969_amd/build.py")
        lib = C.CDLL(LIB_PATH)
        lib.stree_version.restype = C.c_int
        lib.stree_status_string.restype = C.c_char_p
        lib.stree_status_string.argtypes = [C.c_int]
        lib.stree_workspace_bytes.restype = C.c_size_t
        lib.stree_prepare.restype = C.c_int
        lib.stree_prepare.argtypes = []
        lib.stree_workspace_bytes.argtypes = [C.POINTER(StreeDims)]
        dp = C.POINTER(StreeDims)
        lib.stree_tree_index.argtypes = [dp] + [_VP] * 6
        lib.stree_tree_conv.argtypes = [dp] + [_VP] * 8
        lib.stree_tree_ssd.argtypes = [dp] + [_VP] * 11
        lib.stree_commit_state.argtypes = [dp] + [_VP] * 13
        lib.stree_tree_ssd_replay.argtypes = [dp, C.POINTER(StreeReplay)] + [_VP] * 13
        lib.stree_tree_conv_replay.argtypes = [dp, C.POINTER(StreeReplay)] + [_VP] * 11
        lib.stree_tree_step.argtypes = [dp, C.POINTER(StreeReplay)] + [_VP] * 17
        lib.stree_linear_ssd.argtypes = [dp] + [_VP] * 10
        lib.stree_linear_ssd.restype = C.c_int
        lib.stree_gate_norm.argtypes = [dp, _VP, _VP, C.c_int64, _VP, C.c_float, _VP, _VP]
        lib.stree_gate_norm.restype = C.c_int
        for f in (lib.stree_tree_index, lib.stree_tree_conv, lib.stree_tree_ssd, lib.stree_commit_state,
                  lib.stree_tree_ssd_replay, lib.stree_tree_conv_replay, lib.stree_tree_step):
            f.restype = C.c_int
        _lib, _host = lib, None            # (the native half is bound to this library at the first call that needs it)
    return _lib


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()


def _stream() -> int:
    return torch.cuda.current_stream().cuda_stream


def make_dims(batch, nnodes, nheads, headdim, dstate, ngroups, conv_width=0, io_dtype=BF16, flags=0,
              x_stride_n=0, b_stride_n=0, c_stride_n=0, dt_bias: Optional[torch.Tensor] = None,
              state_dtype=F32) -> StreeDims:
    """`dt_bias` (f32 [H] on the GPU) switches the in-kernel softplus on: the dt arguments of the call are
    then the raw projection and the step size is softplus(dt + dt_bias[h])."""
    if dt_bias is not None:
        assert dt_bias.dtype == torch.float32 and dt_bias.is_contiguous() and dt_bias.numel() == nheads
        flags |= FLAG_DT_SOFTPLUS
    return StreeDims(batch, nnodes, nheads, headdim, dstate, ngroups, conv_width, io_dtype, state_dtype, flags,
                     x_stride_n, b_stride_n, c_stride_n, None if dt_bias is None else dt_bias.data_ptr())


def stree_prepare() -> None:
    """Raise, on the current device, the dynamic-LDS limits that two of the kernels otherwise raise at their
    first launch: afterwards every entry point only launches kernels (what a stream capture wants)."""
    _check(load().stree_prepare(), "stree_prepare")


def stree_workspace_bytes(d: StreeDims) -> int:
    """Device scratch the entry points need for these sizes: 0 for every valid shape."""
    return int(load().stree_workspace_bytes(C.byref(d)))


def _check(rc: int, where: str):
    if rc != 0:
        raise StreeError(rc, where)


def stree_tree_index(parent: torch.Tensor, conv_width: int = 4
                     ) -> Tuple[torch.Tensor, torch.Tensor, torch.Tensor, torch.Tensor]:
    """parent int32 [B,N] -> (depth [B,N], ancmask uint32-as-int32 [B,N,ceil(N/32)],
    anc [B,N,W], status [B])."""
    B, N = parent.shape
    dev = parent.device
    depth = torch.empty((B, N), dtype=torch.int32, device=dev)
    mask = torch.empty((B, N, (N + 31) // 32), dtype=torch.int32, device=dev)
    anc = torch.empty((B, N, conv_width), dtype=torch.int32, device=dev)
    status = torch.empty((B,), dtype=torch.int32, device=dev)
    d = make_dims(B, N, 1, 1, 1, 1, conv_width, F32)
    _check(load().stree_tree_index(C.byref(d), _ptr(parent), _ptr(depth), _ptr(mask), _ptr(anc), _ptr(status),
                                   _stream()), "stree_tree_index")
    return depth, mask, anc, status


def stree_tree_conv(parent, xbc_pre, conv_state, conv_w, conv_b, nheads, headdim, dstate, ngroups,
                    silu: bool = True, out: Optional[torch.Tensor] = None, status: Optional[torch.Tensor] = None):
    """xbc_pre [B,N,Cc], conv_state [B,W-1,Cc], conv_w [Cc,W], conv_b [Cc]|None -> xbc_out [B,N,Cc]."""
    return _native().tree_conv(parent, xbc_pre, conv_state, conv_w, conv_b, nheads, headdim, dstate, ngroups, silu, out,
                               status)



def stree_tree_ssd(parent, x, dt, A, Bm, Cm, D=None, h0=None, out: Optional[torch.Tensor] = None,
                   status: Optional[torch.Tensor] = None, force_fma: bool = False, general_mfma: bool = False,
                   dt_bias: Optional[torch.Tensor] = None):
    """x [B,N,H,P], dt [B,N,H] f32, A [H] f32, Bm/Cm [B,N,G,S], D [H]|None, h0 [B,H,P,S] f32 or bf16|None
    -> y [B,N,H,P].  x, Bm, Cm may be column views of one [B,N,Cc] buffer.  With dt_bias [H] f32, dt is
    the raw projection and the kernels take softplus(dt + dt_bias[h]) as the step size (here and in
    every function below that has this argument)."""
    return _native().tree_ssd(parent, x, dt, A, Bm, Cm, D, h0, out, status, force_fma, general_mfma, dt_bias)



def stree_commit_state(parent, accepted, x, dt, A, Bm, h0=None, h_out: Optional[torch.Tensor] = None,
                       xbc_pre=None, conv_state=None, conv_state_out: Optional[torch.Tensor] = None,
                       status: Optional[torch.Tensor] = None, dims: Optional[tuple] = None,
                       dt_bias: Optional[torch.Tensor] = None):
    """-> (h_out [B,H,P,S] in the dtype of h0, conv_state_out [B,W-1,Cc] | None).  h_out may be h0 itself
    (in place), conv_state_out may be conv_state itself.  With x, dt, A, Bm all None only the conv
    tail is updated; `dims` = (H, P, S, G) then names the head shapes."""
    return _native().commit_state(parent, accepted, x, dt, A, Bm, h0, h_out, xbc_pre, conv_state, conv_state_out, status,
                                  dims, dt_bias)



def stree_tree_ssd_replay(prev_parent, prev_accepted, prev_x, prev_dt, prev_Bm, parent, x, dt, A, Bm, Cm, D, h0,
                          h_out: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None,
                          status: Optional[torch.Tensor] = None, replay_status: Optional[torch.Tensor] = None,
                          force_fma: bool = False, dt_bias: Optional[torch.Tensor] = None):
    """Commit of the previous tree's accepted path fused with the scan of the current tree.
    -> (y [B,N,H,P], h_out [B,H,P,S] in the dtype of h0).  h_out may be h0 itself (in place)."""
    return _native().tree_ssd_replay(prev_parent, prev_accepted, prev_x, prev_dt, prev_Bm, parent, x, dt, A, Bm, Cm, D, h0,
                                     h_out, out, status, replay_status, force_fma, dt_bias)



def stree_tree_conv_replay(prev_parent, prev_accepted, prev_xbc_pre, parent, xbc_pre, conv_state, conv_w, conv_b,
                           nheads, headdim, dstate, ngroups, silu: bool = True, out: Optional[torch.Tensor] = None,
                           conv_state_out: Optional[torch.Tensor] = None, status: Optional[torch.Tensor] = None,
                           replay_status: Optional[torch.Tensor] = None):
    """Tree conv seeded by the conv state after the previous tree's accepted path.
    -> (xbc_out [B,N,Cc], conv_state_out [B,W-1,Cc]); conv_state_out must not be conv_state."""
    return _native().tree_conv_replay(prev_parent, prev_accepted, prev_xbc_pre, parent, xbc_pre, conv_state, conv_w, conv_b,
                                      nheads, headdim, dstate, ngroups, silu, out, conv_state_out, status, replay_status)



def stree_tree_step(prev_parent, prev_accepted, prev_xbc_pre, prev_xbc_out, prev_dt, parent, xbc_pre, conv_state,
                    conv_w, conv_b, dt, A, D, h0, nheads, headdim, dstate, ngroups, silu: bool = True,
                    xbc_out: Optional[torch.Tensor] = None, conv_state_out: Optional[torch.Tensor] = None,
                    h_out: Optional[torch.Tensor] = None, out: Optional[torch.Tensor] = None,
                    status: Optional[torch.Tensor] = None, replay_status: Optional[torch.Tensor] = None,
                    force_fma: bool = False, dt_bias: Optional[torch.Tensor] = None):
    """One decoding step in one call: tree conv (seeded by the conv state after the previous tree's
    accepted path), state replay along that path and tree scan.  prev_xbc_out is the previous step's
    conv output [B,Np,Cc] (its x and B columns are replayed; it must not be xbc_out).
    -> (y [B,N,H,P], h_out [B,H,P,S] in the dtype of h0, xbc_out [B,N,Cc], conv_state_out [B,W-1,Cc])."""
    return _native().tree_step(prev_parent, prev_accepted, prev_xbc_pre, prev_xbc_out, prev_dt, parent, xbc_pre, conv_state,
                               conv_w, conv_b, dt, A, D, h0, nheads, headdim, dstate, ngroups, silu, xbc_out, conv_state_out,
                               h_out, out, status, replay_status, force_fma, dt_bias)



def stree_gate_norm(y, z, norm_w, ngroups: int, eps: float = 1e-5, out: Optional[torch.Tensor] = None):
    """Output gate and grouped RMS norm: y [B,N,H,P] dense, z [B,N,H,P] (may be a column view with its
    own token stride), norm_w [H*P] -> out [B,N,H,P]; out may be y itself."""
    return _native().gate_norm(y, z, norm_w, ngroups, eps, out)



def stree_linear_ssd(x, dt, A, Bm, Cm=None, D=None, h0=None, want_y: bool = True,
                     out: Optional[torch.Tensor] = None, h_out: Optional[torch.Tensor] = None,
                     dt_bias: Optional[torch.Tensor] = None):
    """Causal scan of T tokens per sequence: x [B,T,H,P], dt [B,T,H] f32, Bm/Cm [B,T,G,S].
    -> (y [B,T,H,P] or None, h_out [B,H,P,S] in the dtype of h0).  h_out may be h0 itself."""
    return _native().linear_ssd(x, dt, A, Bm, Cm, D, h0, want_y, out, h_out, dt_bias)
