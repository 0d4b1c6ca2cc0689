"""Binding of libmoga.so: argument marshalling only.

Every function has the name and the argument order of its C entry point in
include/moga.h.  torch is used for device memory and for the current HIP stream;
every step of the path runs in the library's kernels.  The calls on tensors go
through `_moga_torch` (csrc/torch_binding.cpp), which allocates outputs and makes
the C call natively; host-only entry points and moga_permute_static go through
ctypes.  There is no fallback: if a library cannot be loaded the first call raises.
"""
from __future__ import annotations

import ctypes
import importlib.machinery
import importlib.util
import os
import threading

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libmoga.so")

MOGA_F32, MOGA_BF16 = 0, 1
(OP_ROUTE, OP_PERMUTE, OP_ATTN_FWD, OP_ATTN_BWD, OP_ROUTE_BWD, OP_BALANCE_LOSS, OP_VARLEN_ATTN_FWD,
 OP_VARLEN_ATTN_BWD, OP_ATTN_BWD_JOINT, OP_ATTN_FWD_CALL, OP_FUSED_ATTN_BWD) = range(11)

_c = ctypes
_vp, _i64, _i32, _f32, _sz = _c.c_void_p, _c.c_int64, _c.c_int, _c.c_float, _c.c_size_t
_SIGNATURES = {
    "moga_status_string": (_c.c_char_p, [_i32]),
    "moga_version": (_i32, []),
    "moga_workspace_bytes": (_sz, [_i32, _i64, _i32, _i32, _i32, _i32, _i32]),
    "moga_workspace_preferred_bytes": (_sz, [_i32, _i64, _i64, _i32, _i32, _i32, _i32, _i32]),
    "moga_route": (_i32, [_vp, _i32, _vp, _vp, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_permute": (_i32, [_vp, _i64, _i32, _vp, _vp, _vp, _i32, _i32, _i32, _vp, _vp, _vp, _vp, _vp,
                            _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_permute_static": (_i32, [_vp, _i64, _i32, _vp, _vp, _vp, _i32, _i32, _i32, _vp, _vp, _vp, _vp,
                                   _vp, _vp, _vp, _vp, _vp]),
    "moga_group_attn_fwd": (_i32, [_vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32, _f32, _vp, _vp,
                                   _vp, _sz, _vp]),
    "moga_group_attn_fwd_ws": (_i32, [_vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32, _f32, _vp, _vp,
                                      _vp, _sz, _vp]),
    "moga_group_attn_fwd_tokens": (_i32, [_vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32, _f32, _vp, _vp, _vp, _vp, _vp,
                                          _vp, _sz, _vp]),
    "moga_unpermute": (_i32, [_vp, _i32, _vp, _vp, _i64, _i32, _i32, _vp, _vp]),
    "moga_unpermute_bwd": (_i32, [_vp, _vp, _i32, _vp, _vp, _i64, _i32, _i32, _vp, _vp, _vp]),
    "moga_group_attn_bwd": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32,
                                   _f32, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_group_attn_bwd_joint": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32,
                                   _f32, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_group_attn_bwd_tokens": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32, _f32, _vp, _vp,
                                          _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_group_attn_bwd_tokens_joint": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _i32, _f32, _vp, _vp,
                                          _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_attn_bwd_status_offset": (_sz, [_i64, _i32]),
    "moga_debug_set_spin_limit": (None, [_i32]),
    "moga_debug_set_small_group_rows": (None, [_i64]),
    "moga_debug_small_calls": (_i32, [_i32, _i32, _vp, _vp, _i32]),
    "moga_debug_attn_blocks": (None, [_i32, _i64, _i64, _i32, _i32, _sz, _vp]),
    "moga_permute_bwd": (_i32, [_vp, _vp, _vp, _i32, _vp, _i64, _i32, _i32, _vp, _vp, _vp, _vp]),
    "moga_route_bwd": (_i32, [_vp, _i32, _vp, _vp, _vp, _vp, _vp, _i64, _i32, _i32, _vp, _vp, _vp,
                              _sz, _vp]),
    "moga_route_bwd_balanced": (_i32, [_vp, _i32, _vp, _vp, _vp, _vp, _vp, _vp, _f32, _f32, _vp, _i64, _i32, _i32, _vp, _vp, _vp,
                                       _sz, _vp]),
    "moga_route_bwd_typed": (_i32, [_vp, _i32, _vp, _vp, _vp, _vp, _vp, _vp, _f32, _f32, _vp, _i64, _i32, _i32, _vp, _vp, _i32, _vp,
                                    _sz, _vp]),
    "moga_fused_attn_fwd": (_i32, [_vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _vp, _vp, _i32, _f32, _vp, _vp, _vp]),
    "moga_fused_attn_bwd": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _i32, _f32,
                                   _vp, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_varlen_attn_fwd": (_i32, [_vp, _vp, _vp, _i32, _i64, _i64, _i32, _i32, _vp, _vp, _i32, _f32, _vp, _vp,
                                    _vp, _sz, _vp]),
    "moga_varlen_attn_bwd": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i64, _i32, _i32, _vp, _vp, _i32,
                                    _f32, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_varlen_attn_bwd_rows": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _i32, _i64, _i64, _i32, _i32, _vp, _vp, _i32,
                                         _f32, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_varlen_attn_fwd_calls": (_i32, [_vp, _i32, _i32, _i32, _i32, _f32, _vp]),
    "moga_varlen_attn_bwd_rows_calls": (_i32, [_vp, _i32, _i32, _i32, _i32, _f32, _vp]),
    "moga_stga_index_sizes": (_i32, [_i32, _i32, _i32, _i32, _i32, _i32, _vp, _i32, _i32, _vp, _vp]),
    "moga_stga_build_index": (_i32, [_i32, _i32, _i32, _i32, _i32, _i32, _vp, _i32, _i32, _vp, _vp, _vp, _vp, _vp,
                                     _vp, _vp]),
    "moga_gather_rows": (_i32, [_vp, _i32, _vp, _i64, _i32, _i32, _vp, _vp]),
    "moga_gather_rows_bwd": (_i32, [_vp, _i32, _vp, _vp, _i64, _i64, _i32, _i32, _i32, _vp, _vp]),
    "moga_gather3_fwd": (_i32, [_vp, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _i64, _vp, _vp, _vp, _vp, _vp, _vp,
                                _vp, _vp, _vp, _vp, _vp]),
    "moga_gather3_bwd": (_i32, [_vp, _vp, _vp, _vp, _vp, _i64, _vp, _vp, _i32, _i64, _i32, _i32, _vp, _vp]),
    "moga_gather3_bwd_qkv": (_i32, [_vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _i64, _vp, _vp, _vp, _vp, _i32, _i64, _i32, _i32,
                                    _vp, _vp, _vp, _vp]),
    "moga_merge3_fwd": (_i32, [_vp, _vp, _vp, _i32, _vp, _vp, _vp, _vp, _i64, _i32, _i32, _vp, _vp]),
    "moga_merge3_bwd": (_i32, [_vp, _vp, _i32, _vp, _vp, _vp, _vp, _i64, _i32, _i32, _vp, _vp, _vp, _vp, _vp]),
    "moga_merge3_bwd_rows": (_i32, [_vp, _vp, _vp, _vp, _i32, _vp, _vp, _vp, _vp, _vp, _vp, _vp, _f32, _i64, _i32, _i32, _vp, _vp, _vp,
                                    _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_balance_loss": (_i32, [_vp, _vp, _i64, _i32, _f32, _vp, _vp, _vp, _vp, _sz, _vp]),
    "moga_balance_loss_bwd": (_i32, [_vp, _vp, _i64, _i32, _f32, _f32, _vp, _i32, _vp, _vp]),
}
EXPORTS = tuple(_SIGNATURES)

_lib = None


class MogaError(RuntimeError):
    def __init__(self, fn, status):
        self.status = status
        super().__init__(f"{fn} failed: {status_string(status)} ({status})")


def load():
    """Load libmoga.so (building it first only if no built library exists)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        from . import build as _build
        _build.build()
    lib = ctypes.CDLL(LIB_PATH)
    for name, (res, args) in _SIGNATURES.items():
        fn = getattr(lib, name)   # AttributeError if an export is missing: fail loudly
        fn.restype, fn.argtypes = res, args
    _lib = lib
    return lib


def status_string(status: int) -> str:
    return load().moga_status_string(int(status)).decode()


def version() -> int:
    return load().moga_version()


def workspace_bytes(op, N, H, D, M, d_model, dtype) -> int:
    return int(load().moga_workspace_bytes(op, N, H, D, M, d_model, dtype))


_nat_lock = threading.Lock()


def _load_native():
    """The native module for this torch (building it first only if none is there)."""
    from . import build as _build
    load()
    path = _build.native_path()
    if not os.path.exists(path):
        _build.build_native()
    name = __package__ + "._moga_torch"
    spec = importlib.util.spec_from_file_location(name, path, loader=importlib.machinery.ExtensionFileLoader(name, path))
    module = importlib.util.module_from_spec(spec)
    spec.loader.exec_module(module)
    return module


class _LazyNative:
    """Stands in for the native module until its first use."""

    def __getattr__(self, name):
        global _nat
        with _nat_lock:
            if _nat is self:
                _nat = _load_native()
        return getattr(_nat, name)


_nat = _LazyNative()


def _st(stream):
    """hipStream_t as an integer, or None for torch's current stream."""
    return None if stream is None else stream.cuda_stream


def _dt(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return MOGA_F32
    if t.dtype == torch.bfloat16:
        return MOGA_BF16
    raise TypeError(f"unsupported dtype {t.dtype}")


def _p(t):
    if t is None:
        return None
    assert t.is_cuda and t.is_contiguous(), "device-resident contiguous tensors only"
    return t.data_ptr()


def _stream(stream):
    return (stream if stream is not None else torch.cuda.current_stream()).cuda_stream


def _check(fn, status):
    if status != 0:
        raise MogaError(fn, status)


def moga_route(x, w, bias=None, want_probs=True, want_logits=False, stream=None):
    """-> (group int32 [N], gate f32 [N], probs f32 [N, M] | None, logits f32 [N, M] | None)"""
    return _nat.route(x, w, bias, want_probs, want_logits, _st(stream))


def moga_permute(group, M, q=None, k=None, v=None, stream=None):
    """-> dict(counts, cu_seqlens, max_seqlen, perm, inv_perm[, qh, kh, vh])"""
    r = _nat.permute(group, M, q, k, v, _st(stream))
    out = {"counts": r[0], "cu_seqlens": r[1], "max_seqlen": r[2], "perm": r[3], "inv_perm": r[4]}
    if q is not None:
        out["qh"], out["kh"], out["vh"] = r[5:]
    return out


def moga_permute_static(group, M, out, q=None, k=None, v=None, stream=None):
    """moga_permute without a workspace and without any allocation, here or in the library:
    `out` holds the caller's tensors counts [M], cu_seqlens [M+1], max_seqlen [1], perm [N],
    inv_perm [N] (and qh, kh, vh [H, N, D] when q, k, v are given); they are written in place."""
    N = group.shape[0]
    H = D = 0
    dt = MOGA_F32
    if q is not None:
        _, H, D = q.shape
        dt = _dt(q)
    st = load().moga_permute_static(_p(group), N, M, _p(q), _p(k), _p(v), dt, H, D, _p(out["counts"]),
                                    _p(out["cu_seqlens"]), _p(out["max_seqlen"]), _p(out["perm"]),
                                    _p(out["inv_perm"]), _p(out.get("qh")), _p(out.get("kh")),
                                    _p(out.get("vh")), _stream(stream))
    _check("moga_permute_static", st)
    return out


def moga_group_attn_fwd(qh, kh, vh, cu_seqlens, softmax_scale, stream=None, out=None, lse=None):
    """-> (oh [H, N, D], lse f32 [H, N])"""
    return _nat.group_attn_fwd(qh, kh, vh, cu_seqlens, softmax_scale, _st(stream), out, lse)


def moga_group_attn_fwd_tokens(qh, kh, vh, cu_seqlens, softmax_scale, perm, gate, stream=None):
    """moga_group_attn_fwd and moga_unpermute in one call -> (oh [H, N, D], lse f32 [H, N], o [N, H, D])"""
    return _nat.group_attn_fwd_tokens(qh, kh, vh, cu_seqlens, softmax_scale, perm, gate, _st(stream))


def moga_unpermute(oh, perm, gate=None, stream=None, out=None):
    """-> o [N, H, D]"""
    return _nat.unpermute(oh, perm, gate, _st(stream), out)


def moga_unpermute_bwd(d_o, oh, perm, gate, stream=None):
    """-> (d_oh [H, N, D], d_gate f32 [N])"""
    return _nat.unpermute_bwd(d_o, oh, perm, gate, _st(stream))


def attn_bwd_status(ws, Nq, H):
    """The int32 status word of a backward workspace (0 after every correct run), as a 1-element view."""
    off = int(load().moga_attn_bwd_status_offset(Nq, H))
    return ws[off:off + 4].view(torch.int32)


def set_small_group_rows(rows: int) -> None:
    """Mean group size below which the bf16 attention calls use their small-group kernels (< 0: defaults)."""
    load().moga_debug_set_small_group_rows(int(rows))


def attn_blocks(op, Nq, Nk, H, M, ws_bytes):
    """(query rows, their last round is split, key rows, theirs is split) of the bf16 attention call's blocks; key rows 0: a forward; 2 for
    the splits: OP_ATTN_BWD_JOINT, OP_FUSED_ATTN_BWD, dQ and dK/dV in one launch of the large-group kernels."""
    out = (ctypes.c_int * 4)()
    load().moga_debug_attn_blocks(op, Nq, Nk, H, M, ws_bytes, out)
    return tuple(out)


def small_calls(op, sizes, H):
    """sizes: (queries, groups) of each of up to three bf16 calls together -> whether it takes the kernels for small groups."""
    n = len(sizes)
    bits = load().moga_debug_small_calls(op, n, (ctypes.c_int64 * n)(*(q for q, _ in sizes)), (ctypes.c_int * n)(*(g for _, g in sizes)), H)
    return tuple(bool(bits >> i & 1) for i in range(n))


def set_spin_limit(polls: int) -> None:
    load().moga_debug_set_spin_limit(int(polls))


def moga_group_attn_bwd(d_oh, qh, kh, vh, oh, lse, cu_seqlens, softmax_scale, stream=None, ws=None):
    """-> (d_qh, d_kh, d_vh) each [H, N, D].  `ws`: the caller's workspace (uint8), else one is allocated."""
    return _nat.group_attn_bwd(d_oh, qh, kh, vh, oh, lse, cu_seqlens, softmax_scale, _st(stream), ws)


def moga_group_attn_bwd_tokens(d_o, qh, kh, vh, oh, lse, cu_seqlens, softmax_scale, perm, gate, want_sorted=True, stream=None):
    """moga_unpermute_bwd, moga_group_attn_bwd and moga_permute_bwd in one call
    -> (d_oh [H, N, D], d_gate f32 [N], d_qh, d_kh, d_vh [H, N, D] | None, d_q, d_k, d_v [N, H, D])"""
    return _nat.group_attn_bwd_tokens(d_o, qh, kh, vh, oh, lse, cu_seqlens, softmax_scale, perm, gate, want_sorted, _st(stream))


def moga_permute_bwd(d_qh, d_kh, d_vh, perm, stream=None):
    """-> (d_q, d_k, d_v) each [N, H, D]"""
    return _nat.permute_bwd(d_qh, d_kh, d_vh, perm, _st(stream))


def moga_route_bwd(x, w, probs, group, gate, d_gate, want_dx=False, stream=None):
    """-> (d_w f32 [M, d_model], d_x f32 [N, d_model] | None)"""
    return _nat.route_bwd(x, w, probs, group, gate, d_gate, want_dx, _st(stream))


def moga_route_bwd_balanced(x, w, probs, group, gate, d_gate, frac, alpha, d_loss, want_dx=False, stream=None):
    """moga_balance_loss_bwd (accumulating; d_loss a device scalar) and moga_route_bwd in one call -> (d_w, d_x | None)"""
    return _nat.route_bwd_balanced(x, w, probs, group, gate, d_gate, frac, alpha, d_loss, want_dx, _st(stream))


def moga_fused_attn_fwd(q, k, v, perm, gate, cu_seqlens, softmax_scale, stream=None):
    """q, k, v [N, H, D] token order -> (o [N, H, D] gated, token order; lse f32 [H, N] sorted order)"""
    return _nat.fused_attn_fwd(q, k, v, perm, gate, cu_seqlens, softmax_scale, _st(stream))


def moga_fused_attn_bwd(d_o, q, k, v, o, lse, perm, inv_perm, gate, cu_seqlens, softmax_scale, stream=None):
    """Token-order tensors -> (d_q, d_k, d_v [N, H, D], d_gate f32 [N])"""
    return _nat.fused_attn_bwd(d_o, q, k, v, o, lse, perm, inv_perm, gate, cu_seqlens, softmax_scale, _st(stream))


def moga_varlen_attn_fwd(qh, kh, vh, cu_seqlens_q, cu_seqlens_k, softmax_scale, stream=None):
    """qh [H, Nq, D]; kh, vh [H, Nk, D] -> (oh [H, Nq, D], lse f32 [H, Nq])"""
    return _nat.varlen_attn_fwd(qh, kh, vh, cu_seqlens_q, cu_seqlens_k, softmax_scale, _st(stream))


def moga_varlen_attn_bwd(d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, softmax_scale, stream=None):
    """-> (d_qh [H, Nq, D], d_kh, d_vh [H, Nk, D])"""
    return _nat.varlen_attn_bwd(d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, softmax_scale, _st(stream))


def moga_varlen_attn_fwd_calls(calls, softmax_scale, stream=None):
    """calls: up to three (qh, kh, vh, cu_seqlens_q, cu_seqlens_k), run together -> [(oh, lse)]"""
    return _nat.varlen_attn_fwd_calls(calls, softmax_scale, _st(stream))


def moga_varlen_attn_bwd_rows_calls(calls, softmax_scale, stream=None):
    """calls: up to three (d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, ws), run together -> [(d_qh, d_kh, d_vh)]"""
    return _nat.varlen_attn_bwd_rows_calls(calls, softmax_scale, _st(stream))


def moga_stga_build_index(T, Hh, Ww, wh, ww, tg, shot_of_frame, a_prev=1, a_next=1, device="cuda"):
    """Static index lists (host builder), uploaded to `device` (None keeps them as numpy arrays)."""
    import numpy as np
    shots = np.ascontiguousarray(np.asarray(shot_of_frame, dtype=np.int32))
    assert shots.shape == (T,)
    G, Nk = ctypes.c_int64(0), ctypes.c_int64(0)
    sp = shots.ctypes.data_as(ctypes.c_void_p)
    st = load().moga_stga_index_sizes(T, Hh, Ww, wh, ww, tg, sp, a_prev, a_next, ctypes.byref(G), ctypes.byref(Nk))
    _check("moga_stga_index_sizes", st)
    N, G, Nk = T * Hh * Ww, G.value, Nk.value
    out = {"q_index": np.empty(N, np.int32), "q_slot": np.empty(N, np.int32), "cu_q": np.empty(G + 1, np.int32),
           "kv_index": np.empty(Nk, np.int32), "cu_k": np.empty(G + 1, np.int32),
           "inv_cu": np.empty(N + 1, np.int32), "inv_slots": np.empty(Nk, np.int32)}
    hp = lambda a: a.ctypes.data_as(ctypes.c_void_p)
    st = load().moga_stga_build_index(T, Hh, Ww, wh, ww, tg, sp, a_prev, a_next, hp(out["q_index"]),
                                      hp(out["q_slot"]), hp(out["cu_q"]), hp(out["kv_index"]), hp(out["cu_k"]),
                                      hp(out["inv_cu"]), hp(out["inv_slots"]))
    _check("moga_stga_build_index", st)
    if device is not None:
        out = {k: torch.from_numpy(v).to(device) for k, v in out.items()}
    out["n_groups"], out["n_keys"] = G, Nk
    return out


def moga_gather_rows(src, index, stream=None):
    """src [N, H, D], index [Nk] -> [H, Nk, D]"""
    return _nat.gather_rows(src, index, _st(stream))


def moga_gather_rows_bwd(d_dst, inv_cu, inv_slots, N, d_src=None, stream=None):
    """d_dst [H, Nk, D] -> d_src [N, H, D]; adds into `d_src` when given."""
    return _nat.gather_rows_bwd(d_dst, inv_cu, inv_slots, N, d_src, _st(stream))


def moga_gather3_fwd(q, k, v, inv_moga, q_slot, inv_cu, inv_slots, inv_frame=None, stream=None):
    """q, k, v [N, H, D] -> (qm, km, vm [H, N, D], qs [H, N, D], ks, vs [H, Nk, D], qf, kf, vf [H, N, D]) in one launch."""
    return _nat.gather3_fwd(q, k, v, inv_moga, q_slot, inv_cu, inv_slots, inv_frame, _st(stream))


def moga_gather3_bwd(g_moga, inv_moga, g_stga, inv_cu, inv_slots, g_frame, inv_frame=None, stream=None):
    """g_moga, g_frame [H, N, D], g_stga [H, Nk, D] -> their token-order sum [N, H, D] (one pass)."""
    return _nat.gather3_bwd(g_moga, inv_moga, g_stga, inv_cu, inv_slots, g_frame, inv_frame, _st(stream))


def moga_gather3_bwd_qkv(g_moga, inv_moga, g_stga, q_slot, inv_cu, inv_slots, g_frame, inv_frame=None, stream=None):
    """g_*: the gradients of q, k and v from a branch -> d_q, d_k, d_v [N, H, D]"""
    return _nat.gather3_bwd_qkv(*g_moga, inv_moga, *g_stga, q_slot, inv_cu, inv_slots, *g_frame, inv_frame, _st(stream))


def moga_merge3_fwd(a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate, stream=None):
    """Three [H, N, D] branch outputs -> their mean [N, H, D] in token order (dynamic branch gated)."""
    return _nat.merge3_fwd(a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate, _st(stream))


def moga_merge3_bwd(d_o, a_moga, inv_moga, inv_stga, inv_frame, gate, stream=None):
    """-> (d_a_moga, d_a_stga, d_a_frame [H, N, D], d_gate f32 [N])"""
    return _nat.merge3_bwd(d_o, a_moga, inv_moga, inv_stga, inv_frame, gate, _st(stream))


def moga_merge3_bwd_rows(d_o, a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate, lse, softmax_scale, cu_moga, cu_q, n_keys,
                         cu_frame, stream=None, room=True):
    """moga_merge3_bwd with the row constants of the three attention backwards; `lse`: those of the three branches
    -> (d_a_moga, d_a_stga, d_a_frame [H, N, D], d_gate f32 [N], three workspaces for moga_varlen_attn_bwd_rows).  room: with what a call
    by itself runs fastest with (34 or 51 MB each, where it splits its last round); calls that run together use what they need."""
    return _nat.merge3_bwd_rows(d_o, a_moga, a_stga, a_frame, inv_moga, inv_stga, inv_frame, gate, *lse, softmax_scale, cu_moga, cu_q,
                                n_keys, cu_frame, room, _st(stream))


def moga_varlen_attn_bwd_rows(d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, softmax_scale, ws, stream=None):
    """moga_varlen_attn_bwd with the row constants already in `ws` (from moga_merge3_bwd_rows)."""
    return _nat.varlen_attn_bwd_rows(d_oh, qh, kh, vh, oh, lse, cu_seqlens_q, cu_seqlens_k, softmax_scale, ws, _st(stream))


def moga_balance_loss(group, gate, M, alpha, stream=None):
    """Eqs. 6-8 -> (loss f32 [1], frac f32 [M], prob f32 [M]), all on the device."""
    return _nat.balance_loss(group, gate, M, alpha, _st(stream))


def moga_balance_loss_bwd(group, frac, alpha, d_loss=1.0, d_gate=None, stream=None):
    """Adds d_loss * dL/d gate to `d_gate` (in place) or returns a new tensor when d_gate is None.
    `d_loss`: a Python number, or a one-element fp32 device tensor (read by the kernel: no host sync)."""
    host, dev = (1.0, d_loss) if isinstance(d_loss, torch.Tensor) else (float(d_loss), None)
    return _nat.balance_loss_bwd(group, frac, alpha, host, dev, d_gate, _st(stream))


def moga_forward(x, w, q, k, v, softmax_scale, want_probs=True, stream=None):
    """Alg. 1 end to end: the forward calls in order on one stream.  Returns a dict."""
    group, gate, probs, _ = moga_route(x, w, want_probs=want_probs, stream=stream)
    pm = moga_permute(group, w.shape[0], q, k, v, stream=stream)
    oh, lse, o = moga_group_attn_fwd_tokens(pm["qh"], pm["kh"], pm["vh"], pm["cu_seqlens"], softmax_scale, pm["perm"], gate,
                                            stream=stream)
    pm.update({"group": group, "gate": gate, "probs": probs, "oh": oh, "lse": lse, "o": o})
    return pm


def moga_backward(fwd, x, w, d_o, softmax_scale, want_dx=False, stream=None):
    """Backward of `moga_forward`: the backward calls in reverse order.  Returns a dict."""
    d_oh, d_gate, d_qh, d_kh, d_vh, d_q, d_k, d_v = moga_group_attn_bwd_tokens(
        d_o, fwd["qh"], fwd["kh"], fwd["vh"], fwd["oh"], fwd["lse"], fwd["cu_seqlens"], softmax_scale, fwd["perm"],
        fwd["gate"], stream=stream)
    d_w, d_x = moga_route_bwd(x, w, fwd["probs"], fwd["group"], fwd["gate"], d_gate, want_dx=want_dx,
                              stream=stream)
    return {"d_q": d_q, "d_k": d_k, "d_v": d_v, "d_w": d_w, "d_x": d_x, "d_gate": d_gate,
            "d_oh": d_oh, "d_qh": d_qh, "d_kh": d_kh, "d_vh": d_vh}


def visual_forward(x, w, q, k, v, softmax_scale, grid, static_index, stream=None):
    """The three-branch attention block of Section 3.2: MoGA (Alg. 1, gated by Eq. 5), the
    spatial-temporal groups of `static_index` (from moga_stga_build_index) and the per-frame groups,
    averaged by moga_merge3_fwd.  Returns a dict with everything the backward needs."""
    T, Hh, Ww = grid
    N = T * Hh * Ww
    si = static_index
    dev = q.device
    group, gate, probs, _ = moga_route(x, w, want_probs=True, stream=stream)
    pm = moga_permute(group, w.shape[0], stream=stream)
    pm["qh"], pm["kh"], pm["vh"], qs, ks, vs, qf, kf, vf = moga_gather3_fwd(q, k, v, pm["inv_perm"], si["q_slot"], si["inv_cu"],
                                                                            si["inv_slots"], stream=stream)
    ident = torch.arange(N + 1, dtype=torch.int32, device=dev)
    cu_f = torch.arange(0, N + 1, Hh * Ww, dtype=torch.int32, device=dev)
    if stream is not None and stream != torch.cuda.current_stream():   # made on the current stream, read on `stream`
        stream.wait_stream(torch.cuda.current_stream())
        for t in (ident, cu_f):
            t.record_stream(stream)
    calls = [(pm["qh"], pm["kh"], pm["vh"], pm["cu_seqlens"], pm["cu_seqlens"]), (qs, ks, vs, si["cu_q"], si["cu_k"]),
             (qf, kf, vf, cu_f, cu_f)]
    (a_m, lse_m), (a_s, lse_s), (a_f, lse_f) = moga_varlen_attn_fwd_calls(calls, softmax_scale, stream=stream)
    o = moga_merge3_fwd(a_m, a_s, a_f, pm["inv_perm"], si["q_slot"], None, gate, stream=stream)
    return {"o": o, "group": group, "gate": gate, "probs": probs, "pm": pm, "a_m": a_m, "lse_m": lse_m,
            "qs": qs, "ks": ks, "vs": vs, "a_s": a_s, "lse_s": lse_s, "qf": qf, "kf": kf, "vf": vf,
            "a_f": a_f, "lse_f": lse_f, "cu_f": cu_f, "ident": ident, "si": si}


def visual_backward(fwd, x, w, d_o, softmax_scale, stream=None):
    """Backward of `visual_forward` -> dict(d_q, d_k, d_v [N, H, D], d_w [M, d_model], d_gate [N])."""
    pm, si = fwd["pm"], fwd["si"]
    # Together the three fill each other's last rounds (2 % at 64 frames x 12 heads, 20 % at 8 x 3).  Of tensors above 2 GiB, whose calls have
    # hundreds of rounds, one at a time.  Either way the most that is held at once is what the gather below reads and writes, nine gradients of rows
    # and three of tokens; together that is held from the attention on, with the row constants.
    together = d_o.numel() * d_o.element_size() <= 2 << 30
    d_m, d_s, d_f, d_gate, ws_m, ws_s, ws_f = moga_merge3_bwd_rows(
        d_o, fwd["a_m"], fwd["a_s"], fwd["a_f"], pm["inv_perm"], si["q_slot"], None, fwd["gate"],
        (fwd["lse_m"], fwd["lse_s"], fwd["lse_f"]), softmax_scale, pm["cu_seqlens"], si["cu_q"], fwd["ks"].shape[1], fwd["cu_f"],
        stream=stream, room=not together)
    calls = [(d_m, pm["qh"], pm["kh"], pm["vh"], fwd["a_m"], fwd["lse_m"], pm["cu_seqlens"], pm["cu_seqlens"], ws_m),
             (d_s, fwd["qs"], fwd["ks"], fwd["vs"], fwd["a_s"], fwd["lse_s"], si["cu_q"], si["cu_k"], ws_s),
             (d_f, fwd["qf"], fwd["kf"], fwd["vf"], fwd["a_f"], fwd["lse_f"], fwd["cu_f"], fwd["cu_f"], ws_f)]
    del d_m, d_s, d_f, ws_m, ws_s, ws_f
    grads = []
    while calls:
        n = len(calls) if together else 1
        grads += moga_varlen_attn_bwd_rows_calls(calls[:n], softmax_scale, stream=stream)
        del calls[:n]
    (dqm, dkm, dvm), (dqs, dks, dvs), (dqf, dkf, dvf) = grads
    del grads
    # every token-order gradient is written once: MoGA rows through inv_perm, the static rows through
    # their slot lists (queries are listed once, keys possibly several times), the frame rows in place
    d_q, d_k, d_v = moga_gather3_bwd_qkv((dqm, dkm, dvm), pm["inv_perm"], (dqs, dks, dvs), si["q_slot"], si["inv_cu"], si["inv_slots"],
                                         (dqf, dkf, dvf), stream=stream)
    del dqm, dkm, dvm, dqs, dks, dvs, dqf, dkf, dvf
    d_w, _ = moga_route_bwd(x, w, fwd["probs"], fwd["group"], fwd["gate"], d_gate, stream=stream)
    return {"d_q": d_q, "d_k": d_k, "d_v": d_v, "d_w": d_w, "d_gate": d_gate}
