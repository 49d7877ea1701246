"""Binding of libstrd.so: same names as the C entry points, torch tensors in and out.

Only marshalling happens: shape checks, output/workspace allocation through torch (device memory
plumbing) and the current HIP stream -- in the extension module strd_host (csrc/host.cpp) for the
calls of a layer, where the host's time per call counts, and through ctypes here for the rest.  Every
step of the path runs in the library's kernels; if a library is missing the first call fails loudly.
"""
from __future__ import annotations

import ctypes
import importlib.util
import os
from typing import Optional, Sequence, Tuple

import torch

LIB_PATH = os.path.join(os.path.dirname(os.path.abspath(__file__)), "libstrd.so")

STRD_F32, STRD_BF16 = 0, 1
_c = ctypes
_vp, _int, _i64, _f32, _sz = _c.c_void_p, _c.c_int, _c.c_int64, _c.c_float, _c.c_size_t

_SIGNATURES = {
    "strd_status_string": (_c.c_char_p, [_int]),
    "strd_version": (_int, []),
    "strd_score_attn_kernel_path": (_int, [_int] * 6),
    "strd_score_mamba_kernel_path": (_int, [_int] * 6),
    "strd_ssd_prefill_kernel_path": (_int, [_int] * 6),
    "strd_attn_prefill_kernel_path": (_int, [_int] * 5),
    "strd_score_attn_workspace": (_sz, [_int] * 5 + [_int]),
    "strd_score_attn": (_int, [_vp, _vp, _vp] + [_int] * 5 + [_f32, _int, _vp, _sz, _vp]),
    "strd_score_mamba_workspace": (_sz, [_int] * 5 + [_int]),
    "strd_score_mamba": (_int, [_vp, _vp, _vp, _vp] + [_int] * 5 + [_int, _vp, _sz, _vp]),
    "strd_score_mamba_full_workspace": (_sz, [_int] * 5 + [_int]),
    "strd_score_mamba_full": (_int, [_vp] * 5 + [_int] * 5 + [_int, _vp, _sz, _vp]),
    "strd_select_topk_workspace": (_sz, [_int, _int]),
    "strd_select_topk": (_int, [_vp, _int, _int, _vp, _vp, _sz, _vp]),
    "strd_select_topk_noalloc_max_n": (_int, []),
    "strd_select_topk_noalloc": (_int, [_vp, _int, _int, _vp, _vp]),
    "strd_compact": (_int, [_vp, _vp, _vp, _int, _int, _int, _i64, _vp, _vp, _vp]),
    "strd_compact_batch": (_int, [_vp, _int, _vp, _int, _int, _int, _vp, _vp, _vp]),
    "strd_mfma_rate_probe": (_int, [_vp, _int, _int, _int, _vp]),
    "strd_score_attn_varlen_workspace": (_sz, [_vp, _int, _int, _int, _int, _int]),
    "strd_score_attn_varlen": (_int, [_vp, _vp, _vp, _int, _vp, _int, _int, _int, _int, _f32, _int, _vp, _sz, _vp]),
    "strd_score_attn_varlen_padded": (_int, [_vp, _vp, _vp, _int, _vp, _int, _int, _int, _int, _f32, _int, _vp, _sz, _vp]),
    "strd_score_mamba_varlen_workspace": (_sz, [_vp, _int, _int, _int, _int, _int]),
    "strd_score_mamba_varlen": (_int, [_vp, _vp, _vp, _vp, _int, _vp, _int, _int, _int, _int, _int, _vp, _sz, _vp]),
    "strd_score_mamba_varlen_padded": (_int, [_vp, _vp, _vp, _vp, _int, _vp, _int, _int, _int, _int, _int, _vp, _sz, _vp]),
    "strd_select_topk_varlen_max_n": (_int, []),
    "strd_select_topk_varlen": (_int, [_vp, _int, _vp, _int, _vp, _vp]),
    "strd_compact_varlen": (_int, [_vp, _int, _vp, _vp, _int, _vp, _vp, _vp]),
    "strd_ssd_prefill_workspace": (_sz, [_int] * 6 + [_int]),
    "strd_ssd_prefill": (_int, [_vp] * 9 + [_int] * 6 + [_int, _vp, _sz, _vp]),
    "strd_ssd_prefill_gather": (_int, [_vp] * 10 + [_int] * 8 + [_int, _vp, _sz, _vp]),
    "strd_attn_prefill_workspace": (_sz, [_int] * 4 + [_int]),
    "strd_attn_prefill": (_int, [_vp] * 4 + [_int] * 4 + [_f32, _int, _vp, _sz, _vp]),
    "strd_linear": (_int, [_vp, _vp, _vp, _vp, _int, _int, _int, _int, _vp]),
    "strd_linear_mfma": (_int, [_vp, _vp, _vp, _vp, _int, _int, _int, _int, _vp]),
    "strd_linear_library": (_int, [_vp, _vp, _vp, _vp, _int, _int, _int, _int, _vp]),
    "strd_linear_mfma_supported": (_int, [_int, _int, _int, _int]),
    "strd_linear_mfma_cut": (_int, [_int, _int]),
    "strd_rmsnorm": (_int, [_vp, _vp, _vp, _int, _int, _f32, _int, _vp]),
    "strd_gated_rmsnorm": (_int, [_vp, _vp, _int, _vp, _vp, _int, _int, _int, _f32, _int, _vp]),
    "strd_conv1d_silu": (_int, [_vp, _int, _vp, _vp, _vp, _vp, _vp] + [_int] * 4 + [_int, _vp]),
    "strd_softplus_dt": (_int, [_vp, _int, _int, _vp, _vp, _int, _int, _int, _vp]),
    "strd_avgpool": (_int, [_vp, _vp, _int, _int, _int, _int, _int, _vp, _vp, _vp]),
    "strd_ssd_decode_step": (_int, [_vp] * 8 + [_int] * 4 + [_int, _vp]),
    "strd_attn_decode_step_workspace": (_c.c_size_t, [_int, _int, _int, _int, _int]),
    "strd_attn_decode_step": (_int, [_vp, _vp, _vp, _vp, _int, _int, _int, _int, _f32, _int, _vp, _c.c_size_t, _vp]),
    "strd_schedule_budgets": (_int, [_vp, _int, _int, _int, _vp]),
    "strd_schedule_sigmoid": (_int, [_int, _c.c_double, _c.c_double, _c.c_double, _c.c_double, _vp]),
    "strd_schedule_step_decay": (_int, [_vp, _vp, _vp, _int, _int, _vp]),
    "strd_hybrid_layout": (_int, [_int, _vp]),
    "strd_schedule_named": (_int, [_c.c_char_p, _vp]),
}

_lib = None


class StrdError(RuntimeError):
    pass


def lib():
    """The loaded C library (raises if it has not been built)."""
    global _lib
    if _lib is None:
        if not os.path.exists(LIB_PATH):
            raise StrdError("%s is missing: run `python -m paper_2603_00198_amd.build` "
                            "(there is no fallback path)" % LIB_PATH)
        L = ctypes.CDLL(LIB_PATH)
        for name, (res, args) in _SIGNATURES.items():
            fn = getattr(L, name)
            fn.restype, fn.argtypes = res, args
        _lib = L
    return _lib


_host = None


def host():
    """The extension module that marshals the calls of a layer (raises if it has not been built)."""
    global _host
    if _host is None:
        lib()
        path = os.path.join(os.path.dirname(os.path.abspath(__file__)), "strd_host.so")
        if not os.path.exists(path):
            raise StrdError("%s is missing: run `python -m paper_2603_00198_amd.build`" % path)
        spec = importlib.util.spec_from_file_location("strd_host", path)
        mod = importlib.util.module_from_spec(spec)
        spec.loader.exec_module(mod)
        mod.set_error(StrdError)
        _host = mod
    return _host


def exported_symbols() -> Sequence[str]:
    return tuple(_SIGNATURES)


PATH_NONE, PATH_MFMA, PATH_SIMT = 0, 1, 2


def kernel_path(op: str, *sizes: int, dtype: torch.dtype = torch.bfloat16) -> int:
    """PATH_MFMA / PATH_SIMT / PATH_NONE for op in {"score_attn", "score_mamba", "ssd_prefill",
    "attn_prefill"} with the size arguments of that entry point (host only)."""
    io = STRD_BF16 if dtype == torch.bfloat16 else STRD_F32
    return getattr(lib(), "strd_%s_kernel_path" % op)(*[int(v) for v in sizes], io)


def _check(rc: int, what: str):
    if rc != 0:
        raise StrdError("%s failed: %s" % (what, lib().strd_status_string(rc).decode()))


def _io(t: torch.Tensor) -> int:
    if t.dtype == torch.float32:
        return STRD_F32
    if t.dtype == torch.bfloat16:
        return STRD_BF16
    raise StrdError("unsupported tensor dtype %s (fp32 or bf16)" % t.dtype)


def _dev(*ts: Optional[torch.Tensor]):
    for t in ts:
        if t is None:
            continue
        if not t.is_cuda:
            raise StrdError("tensors must live on the GPU")
        if not t.is_contiguous():
            raise StrdError("tensors must be contiguous")


def _ptr(t: Optional[torch.Tensor]):
    return None if t is None else t.data_ptr()


def _stream():
    return torch.cuda.current_stream().cuda_stream


def _ws(nbytes: int, like: torch.Tensor) -> Tuple[Optional[torch.Tensor], int]:
    if nbytes == 0:
        return None, 0
    return torch.empty(nbytes, dtype=torch.uint8, device=like.device), nbytes


def score_attn(q_txt: torch.Tensor, k_vis: torch.Tensor, scale: Optional[float] = None,
               out: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """s[N] fp32 from text queries [M,Hq,d] and vision keys [N,Hkv,d]."""
    return (_host or host()).score_attn(q_txt, k_vis, scale, out, ws)


def score_mamba(B_vis: torch.Tensor, C_txt: torch.Tensor, dt_vis: torch.Tensor,
                out: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """s[N] fp32 from vision b [N,G,n], text c [M,G,n] and vision dt [N,H] (fp32)."""
    return (_host or host()).score_mamba(B_vis, C_txt, dt_vis, out, ws)


def score_mamba_full(B_vis: torch.Tensor, C_txt: torch.Tensor, dt_all: torch.Tensor, A: torch.Tensor,
                     out: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Full Mamba Dynamic score s[N] fp32 from vision b [N,G,n], text c [M,G,n], dt of all tokens
    [N+M,H] (fp32, vision rows first) and A [H]."""
    _dev(B_vis, C_txt, dt_all, A, out, ws)
    N, G, n = B_vis.shape
    M = C_txt.shape[0]
    H = dt_all.shape[1]
    if C_txt.shape[1:] != (G, n) or dt_all.shape[0] != N + M or dt_all.dtype != torch.float32 \
            or A.shape != (H,) or A.dtype != torch.float32 or B_vis.dtype != C_txt.dtype:
        raise StrdError("B/C/dt/A mismatch")
    io = _io(B_vis)
    if out is None:
        out = torch.empty(N, dtype=torch.float32, device=B_vis.device)
    need = lib().strd_score_mamba_full_workspace(M, N, H, G, n, io)
    if ws is None:
        ws, _ = _ws(need, B_vis)
    _check(lib().strd_score_mamba_full(_ptr(B_vis), _ptr(C_txt), _ptr(dt_all), _ptr(A), _ptr(out), M, N, H, G, n, io,
                                       _ptr(ws), 0 if ws is None else ws.numel(), _stream()), "score_mamba_full")
    return out


def select_topk(scores: torch.Tensor, K: int, out: Optional[torch.Tensor] = None,
                ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """idx[K] int32 ascending: the K highest scores, ties to the lowest index."""
    return (_host or host()).select_topk(scores, K, out, ws)


def select_topk_noalloc(scores: torch.Tensor, K: int, out: torch.Tensor) -> torch.Tensor:
    """select_topk through the entry point that allocates nothing: `out` [K] int32 is the caller's."""
    _dev(scores, out)
    if scores.dtype != torch.float32 or scores.dim() != 1 or out.dtype != torch.int32 or out.shape != (K,):
        raise StrdError("scores must be a 1-D fp32 tensor, out a [K] int32 tensor")
    _check(lib().strd_select_topk_noalloc(_ptr(scores), scores.shape[0], K, _ptr(out), _stream()), "select_topk_noalloc")
    return out


def compact(src: Optional[torch.Tensor], idx: torch.Tensor, N: int, M: int,
            pos_in: Optional[torch.Tensor] = None, want_pos: bool = False,
            out: Optional[torch.Tensor] = None):
    """Gather rows idx (vision) + the M text rows of src [N+M, ...]; returns dst or (dst, pos_out)."""
    _dev(src, idx, pos_in, out)
    if idx.dtype != torch.int32:
        raise StrdError("idx must be int32")
    K = idx.shape[0]
    dst, row_bytes = None, 0
    if src is not None:
        if src.shape[0] != N + M:
            raise StrdError("src must have N+M rows")
        row_bytes = (src.numel() // max(src.shape[0], 1)) * src.element_size() if src.shape[0] else 0
        if src.shape[0] == 0:
            row_bytes = int(torch.Size(src.shape[1:]).numel()) * src.element_size()
        dst = out if out is not None else torch.empty((K + M,) + tuple(src.shape[1:]), dtype=src.dtype,
                                                      device=src.device)
    pos_out = None
    if want_pos or pos_in is not None:
        pos_out = torch.empty(K + M, dtype=torch.int32, device=idx.device)
    _check(lib().strd_compact(_ptr(src), _ptr(idx), _ptr(dst), N, M, K, row_bytes, _ptr(pos_in), _ptr(pos_out),
                              _stream()), "compact")
    if pos_out is not None:
        return dst, pos_out
    return dst


class _CompactItem(ctypes.Structure):
    _fields_ = [("src", _vp), ("dst", _vp), ("row_bytes", _i64)]


def compact_batch(srcs: Sequence[torch.Tensor], idx: torch.Tensor, N: int, M: int,
                  pos_in: Optional[torch.Tensor] = None, want_pos: bool = False,
                  outs: Optional[Sequence[torch.Tensor]] = None):
    """One-launch gather of several [N+M, ...] tensors by the same idx; returns (dsts, pos_out or None)."""
    return (_host or host()).compact_batch(srcs, idx, N, M, pos_in, want_pos, outs)


def mfma_rate_probe(workgroups: int, iters: int, random_operands: bool, out: Optional[torch.Tensor] = None,
                    device="cuda", small_products: bool = False) -> torch.Tensor:
    """Launches the matrix-core rate probe (a measurement aid): workgroups * 4 * iters * 32 * 32768 flop, as
    32 x 32 x 16 products or (small_products) twice as many 16 x 16 x 32 ones."""
    if out is None:
        out = torch.empty(workgroups * 256, dtype=torch.float32, device=device)
    _dev(out)
    mode = int(bool(random_operands)) | (2 if small_products else 0)
    _check(lib().strd_mfma_rate_probe(_ptr(out), workgroups, iters, mode, _stream()), "mfma_rate_probe")
    return out


# ---- packed batches of sequences: `seqs` is a list of (N, M, K) per sequence ----------------
class _Seq(ctypes.Structure):
    _fields_ = [("N", ctypes.c_int32), ("M", ctypes.c_int32), ("K", ctypes.c_int32)]


def score_attn_varlen(q_all: torch.Tensor, k_all: torch.Tensor, seqs, scale: Optional[float] = None,
                      ld: Optional[int] = None, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """scores [nseq, ld] fp32 of a packed batch: q_all [rows,Hq,d], k_all [rows,Hkv,d]."""
    return (_host or host()).score_attn_varlen(q_all, k_all, seqs, scale, ld, out)


def score_mamba_varlen(B_all: torch.Tensor, C_all: torch.Tensor, dt_all: torch.Tensor, seqs,
                       ld: Optional[int] = None, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """scores [nseq, ld] fp32 of a packed batch: B_all, C_all [rows,G,n], dt_all [rows,H] fp32."""
    return (_host or host()).score_mamba_varlen(B_all, C_all, dt_all, seqs, ld, out)


def select_topk_varlen(scores: torch.Tensor, seqs, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """idx [sum K] int32: per sequence, the K_b best of scores[b, :N_b], ascending, local to the sequence."""
    return (_host or host()).select_topk_varlen(scores, seqs, out)


def compact_varlen(srcs: Sequence[torch.Tensor], idx: torch.Tensor, seqs, pos_in: Optional[torch.Tensor] = None,
                   want_pos: bool = False):
    """One-launch gather of several packed [rows, ...] tensors; returns (dsts [sum(K+M), ...], pos_out or None)."""
    return (_host or host()).compact_varlen(srcs, idx, seqs, pos_in, want_pos)


def ssd_prefill(x: torch.Tensor, dt: torch.Tensor, A: torch.Tensor, B: torch.Tensor, C: torch.Tensor,
                D: Optional[torch.Tensor] = None, S_in: Optional[torch.Tensor] = None, chunk: int = 256,
                want_state: bool = True, out: Optional[torch.Tensor] = None,
                ws: Optional[torch.Tensor] = None):
    """Mamba-2 scan: returns (y [T,H,P], S_out [H,P,n] fp32 or None)."""
    return (_host or host()).ssd_prefill(x, dt, A, B, C, D, S_in, chunk, want_state, out, ws)


def ssd_prefill_gather(x: torch.Tensor, dt: torch.Tensor, A: torch.Tensor, B: torch.Tensor, C: torch.Tensor,
                       idx: torch.Tensor, N: int, M: int, D: Optional[torch.Tensor] = None,
                       S_in: Optional[torch.Tensor] = None, chunk: int = 256, want_state: bool = True,
                       out: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None):
    """Mamba-2 scan over rows idx (vision) + the M text rows of the uncompacted inputs [N+M, ...]."""
    return (_host or host()).ssd_prefill_gather(x, dt, A, B, C, idx, N, M, D, S_in, chunk, want_state, out, ws)


def attn_prefill(q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, scale: Optional[float] = None,
                 out: Optional[torch.Tensor] = None, ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """Causal GQA attention: o [T,Hq,d]."""
    return (_host or host()).attn_prefill(q, k, v, scale, out, ws)


def avgpool(src: torch.Tensor, N: int, M: int, K: int, pos_in: Optional[torch.Tensor] = None,
            want_pos: bool = False):
    """Average-pool the N vision rows of src [N+M, D] into K consecutive windows, keep the M text
    rows; returns dst [K+M, D] or (dst, pos_out)."""
    _dev(src, pos_in)
    if src.dim() != 2 or src.shape[0] != N + M:
        raise StrdError("avgpool: src must be [N+M, D]")
    dst = torch.empty((K + M, src.shape[1]), dtype=src.dtype, device=src.device)
    pos = torch.empty(K + M, dtype=torch.int32, device=src.device) if (want_pos or pos_in is not None) else None
    _check(lib().strd_avgpool(_ptr(src), _ptr(dst), N, M, K, src.shape[1], _io(src), _ptr(pos_in), _ptr(pos),
                              _stream()), "avgpool")
    return (dst, pos) if pos is not None else dst


def ssd_decode_step(x: torch.Tensor, dt: torch.Tensor, A: torch.Tensor, B: torch.Tensor, C: torch.Tensor,
                    D: Optional[torch.Tensor], S: torch.Tensor) -> torch.Tensor:
    """One token of the recurrence: x [H,P], dt [H] fp32, B, C [G,n], S [H,P,n] fp32 updated in
    place; returns y [H,P]."""
    return (_host or host()).ssd_decode_step(x, dt, A, B, C, D, S)


def attn_decode_step(q: torch.Tensor, k_cache: torch.Tensor, v_cache: torch.Tensor, scale: Optional[float] = None,
                     ws: Optional[torch.Tensor] = None) -> torch.Tensor:
    """The newest token's attention over the T cached rows (its own included): q [Hq,d],
    k_cache, v_cache [T,Hkv,d]; returns o [Hq,d]."""
    return (_host or host()).attn_decode_step(q, k_cache, v_cache, scale, ws)


def schedule_budgets(alpha: Sequence[float], N0: int, K_min: int = 0):
    """Per-layer budgets K_l from retention ratios alpha_l (host only)."""
    L = len(alpha)
    a = (ctypes.c_double * L)(*[float(v) for v in alpha])
    k = (ctypes.c_int32 * L)()
    _check(lib().strd_schedule_budgets(ctypes.cast(a, _vp), L, int(N0), int(K_min), ctypes.cast(k, _vp)),
           "schedule_budgets")
    return list(k)


def schedule_sigmoid(L: int, a_start: float = 1.0, a_end: float = 0.125, k: float = 20.0, x0: float = 0.11):
    """Sigmoid retention ratios alpha_l, l = 0..L-1 (host only)."""
    out = (ctypes.c_double * L)()
    _check(lib().strd_schedule_sigmoid(int(L), a_start, a_end, k, x0, ctypes.cast(out, _vp)), "schedule_sigmoid")
    return list(out)


# ------------------------------------------------------------------ block glue -------------
def linear(x: torch.Tensor, w: torch.Tensor, residual: Optional[torch.Tensor] = None,
           out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """x [T,Kd] . w [Kd,Nd] (+ residual [T,Nd]): the library's own kernel for large bf16 products, rocBLAS otherwise."""
    return (_host or host()).linear(x, w, residual, out)


def _linear_by(entry: str, x, w, residual, out):
    _dev(x, w, residual, out)
    T, Kd = x.shape
    Nd = w.shape[1]
    if w.shape[0] != Kd or w.dtype != x.dtype or (residual is not None and (residual.shape != (T, Nd) or
                                                                             residual.dtype != x.dtype)):
        raise StrdError("%s: x [T,Kd], w [Kd,Nd], residual [T,Nd], one dtype" % entry)
    out = out if out is not None else torch.empty((T, Nd), dtype=x.dtype, device=x.device)
    _check(getattr(lib(), "strd_" + entry)(_ptr(x), _ptr(w), _ptr(residual), _ptr(out), T, Kd, Nd, _io(x), _stream()), entry)
    return out


def linear_mfma(x: torch.Tensor, w: torch.Tensor, residual: Optional[torch.Tensor] = None,
                out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """The same product by the library's own matrix-core kernel only (bf16; no handle, no allocation)."""
    return _linear_by("linear_mfma", x, w, residual, out)


def linear_library(x: torch.Tensor, w: torch.Tensor, residual: Optional[torch.Tensor] = None,
                   out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """The same product by rocBLAS whatever the shape (to time the two side by side)."""
    return _linear_by("linear_library", x, w, residual, out)


def linear_mfma_supported(T: int, Kd: int, Nd: int, dtype: torch.dtype) -> bool:
    return bool(lib().strd_linear_mfma_supported(T, Kd, Nd, 1 if dtype == torch.bfloat16 else 0))


def rmsnorm(x: torch.Tensor, w: torch.Tensor, eps: float = 1e-5, out: Optional[torch.Tensor] = None) -> torch.Tensor:
    return (_host or host()).rmsnorm(x, w, eps, out)


def gated_rmsnorm(y: torch.Tensor, z: torch.Tensor, w: torch.Tensor, groups: int = 1, eps: float = 1e-5,
                  out: Optional[torch.Tensor] = None) -> torch.Tensor:
    """rmsnorm(y * silu(z)) * w per group of channels; z may be a column slice of a wider matrix."""
    return (_host or host()).gated_rmsnorm(y, z, w, groups, eps, out)


def conv1d_silu(xbc: torch.Tensor, w: torch.Tensor, b: Optional[torch.Tensor], Cx: int, Cb: int):
    """Causal depthwise conv (w [Cx+2Cb, W]) + SiLU over the first Cx+2Cb columns of xbc (may be a
    column slice); returns contiguous x [T,Cx], B [T,Cb], C [T,Cb]."""
    return (_host or host()).conv1d_silu(xbc, w, b, Cx, Cb)


def softplus_dt(raw: torch.Tensor, bias: Optional[torch.Tensor] = None) -> torch.Tensor:
    """dt [T,H] fp32 = softplus(raw + bias); raw [T,H] may be a column slice, bias [H] fp32."""
    return (_host or host()).softplus_dt(raw, bias)


HYBRID_LAYERS = 62
LAYER_MAMBA, LAYER_MLP, LAYER_ATTN = 0, 1, 2
NAMED_SCHEDULES = ("attn_only_1st_attn", "all_attn_25", "all_attn_35", "all_attn_50", "first_mamba", "second_mamba",
                   "all_attn_1m", "all_attn_2m", "sigmoid_25", "sigmoid_35", "sigmoid_50")


def schedule_step_decay(ranges: Sequence[Tuple[int, int, float]], L: int):
    """alpha_l from (lo, hi, alpha) ranges (inclusive, later ranges win; 1.0 elsewhere)."""
    n = len(ranges)
    lo = (ctypes.c_int * n)(*[int(r[0]) for r in ranges])
    hi = (ctypes.c_int * n)(*[int(r[1]) for r in ranges])
    al = (ctypes.c_double * n)(*[float(r[2]) for r in ranges])
    out = (ctypes.c_double * L)()
    _check(lib().strd_schedule_step_decay(ctypes.cast(lo, _vp), ctypes.cast(hi, _vp), ctypes.cast(al, _vp), n, int(L),
                                          ctypes.cast(out, _vp)), "schedule_step_decay")
    return list(out)


def hybrid_layout(L: int = HYBRID_LAYERS):
    """Layer types (LAYER_MAMBA / LAYER_MLP / LAYER_ATTN) of the 62-layer hybrid of the paper's schedules."""
    out = (ctypes.c_int32 * L)()
    _check(lib().strd_hybrid_layout(int(L), ctypes.cast(out, _vp)), "hybrid_layout")
    return list(out)


def schedule_named(name: str):
    """Retention ratios of one of NAMED_SCHEDULES for the 62 layers."""
    out = (ctypes.c_double * HYBRID_LAYERS)()
    _check(lib().strd_schedule_named(name.encode(), ctypes.cast(out, _vp)), "schedule_named(%s)" % name)
    return list(out)
