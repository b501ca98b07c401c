"""ctypes binding with the same names as the C ABI (include/antkv.h).  Argument marshalling only."""
from __future__ import annotations

import ctypes
import functools
import os
from dataclasses import dataclass

import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libantkv.so")
_lib = None

EXPORTS = (
    "antkv_version", "antkv_strerror", "antkv_encode", "antkv_anchor_select_workspace", "antkv_anchor_select",
    "antkv_topk_workspace", "antkv_topk", "antkv_gather_rows", "antkv_decode_attn_workspace", "antkv_decode_attn",
    "antkv_decode_attn_static", "antkv_set_decode_options", "antkv_decode_attn_prerope_workspace", "antkv_decode_attn_prerope", "antkv_append_token", "antkv_prefill_attn", "antkv_kmeans_step_workspace", "antkv_kmeans_step",
)


class AntkvError(RuntimeError):
    def __init__(self, code: int, what: str):
        super().__init__(f"{what}: error {code} ({_strerror(code)})")
        self.code = code


class _Geom(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("B", "Hq", "Hkv", "D", "d_sub", "n_centroids")]


@dataclass(frozen=True)
class Geometry:
    B: int
    Hq: int
    Hkv: int
    d_sub: int
    D: int = 128
    n_centroids: int = 256

    @property
    def M(self) -> int:
        return self.D // self.d_sub

    @property
    def code_bytes(self) -> int:
        """Bytes of one token's codes: one byte per sub-space, or the M 12-bit codes packed (4096 centroids)."""
        return self.M if self.n_centroids <= 256 else (self.M * 12 + 7) // 8

    def c(self) -> _Geom:
        return _Geom(self.B, self.Hq, self.Hkv, self.D, self.d_sub, self.n_centroids)

    @functools.cached_property
    def _c(self) -> _Geom:
        """Built on first use: a call passes it by reference and only reads it."""
        return self.c()


def lib_path() -> str:
    return _LIB_PATH


def load_library():
    """Load libantkv.so; fails loudly if it has not been built (there is no fallback path)."""
    global _lib
    if _lib is None:
        if not os.path.exists(_LIB_PATH):
            raise ImportError(f"{_LIB_PATH} is missing: build it with `python -m paper_2506_19505_amd.build` "
                              "(or __graft_entry__.build()); the AnTKV path has no CPU fallback")
        lib = ctypes.CDLL(_LIB_PATH)
        i64, vp, sz, f32 = ctypes.c_int64, ctypes.c_void_p, ctypes.c_size_t, ctypes.c_float
        gp = ctypes.POINTER(_Geom)
        lib.antkv_version.restype = ctypes.c_int
        lib.antkv_strerror.restype = ctypes.c_char_p
        lib.antkv_strerror.argtypes = [ctypes.c_int]
        lib.antkv_encode.restype = ctypes.c_int
        lib.antkv_encode.argtypes = [gp, vp, i64, i64, i64, i64, vp, vp, i64, i64, vp]
        lib.antkv_anchor_select_workspace.restype = sz
        lib.antkv_anchor_select_workspace.argtypes = [gp, i64, i64, i64]
        lib.antkv_anchor_select.restype = ctypes.c_int
        lib.antkv_anchor_select.argtypes = [gp, vp, vp, i64, i64, f32, i64, vp, vp, vp, vp, vp, vp, vp, sz, vp]
        lib.antkv_topk_workspace.restype = sz
        lib.antkv_topk_workspace.argtypes = [i64, i64, i64]
        lib.antkv_topk.restype = ctypes.c_int
        lib.antkv_topk.argtypes = [vp, i64, i64, i64, vp, vp, sz, vp]
        lib.antkv_gather_rows.restype = ctypes.c_int
        lib.antkv_gather_rows.argtypes = [gp, vp, i64, vp, i64, vp, vp]
        lib.antkv_kmeans_step_workspace.restype = sz
        lib.antkv_kmeans_step_workspace.argtypes = [gp]
        lib.antkv_kmeans_step.restype = ctypes.c_int
        lib.antkv_kmeans_step.argtypes = [gp, vp, vp, i64, vp, vp, vp, vp, vp, vp, sz, vp]
        lib.antkv_prefill_attn.restype = ctypes.c_int
        lib.antkv_prefill_attn.argtypes = [gp, vp, vp, vp, i64, i64, f32, vp, vp, vp, vp]
        lib.antkv_append_token.restype = ctypes.c_int
        lib.antkv_append_token.argtypes = [gp, vp, vp, i64, i64, vp, vp, vp, vp, i64, vp, vp, i64, vp, vp, i64, vp]
        lib.antkv_decode_attn_workspace.restype = sz
        lib.antkv_decode_attn_workspace.argtypes = [gp, i64, i64, i64, i64]
        lib.antkv_decode_attn.restype = ctypes.c_int
        lib.antkv_decode_attn.argtypes = [gp, vp, f32, vp, vp, i64, i64, vp, vp, vp, vp, i64, vp, vp, i64, vp,
                                          vp, vp, vp, vp, i64, vp, sz, vp]
        lib.antkv_decode_attn_static.restype = ctypes.c_int
        lib.antkv_decode_attn_static.argtypes = [gp, vp, f32, vp, vp, i64, i64, vp, vp, vp, vp, i64, vp, vp, i64, vp, vp]
        lib.antkv_set_decode_options.restype = ctypes.c_int
        lib.antkv_set_decode_options.argtypes = [ctypes.c_int]
        lib.antkv_decode_attn_prerope_workspace.restype = sz
        lib.antkv_decode_attn_prerope_workspace.argtypes = [gp, i64, i64]
        lib.antkv_decode_attn_prerope.restype = ctypes.c_int
        lib.antkv_decode_attn_prerope.argtypes = [gp, vp, f32, vp, vp, i64, i64, vp, vp, vp, vp, i64, vp, vp, i64,
                                                  f32, ctypes.c_int, i64, vp, vp, sz, vp]
        _lib = lib
    return _lib


def _strerror(code: int) -> str:
    return load_library().antkv_strerror(code).decode()


def version() -> int:
    return int(load_library().antkv_version())


# Host cost of a call: argument conversion, the stream and the checks took 6 us of the 9.5 us of a decode_attn call when
# every argument became a c_void_p and the stream came through torch.cuda.current_stream (2 us by itself).  Addresses go as
# plain ints (ctypes converts them by argtypes) and the stream's handle is asked for directly: 5 us, launch included.
def _p(t):
    return None if t is None else t.data_ptr()


def _stream(t: torch.Tensor):
    return torch._C._cuda_getCurrentRawStream(t.get_device())


def _check(rc: int, what: str):
    if rc != 0:
        raise AntkvError(rc, what)


def _need(t: torch.Tensor, dtype, name: str):
    if t.is_cuda and t.dtype is dtype and t.is_contiguous():
        return
    if not t.is_cuda:
        raise ValueError(f"{name} must be a device tensor")
    if t.dtype != dtype:
        raise TypeError(f"{name} must be {dtype}")
    if not t.is_contiguous():
        raise ValueError(f"{name} must be contiguous")


def _workspace(nbytes: int, device) -> torch.Tensor:
    return torch.empty(max(int(nbytes), 256), dtype=torch.uint8, device=device)


def encode(geom: Geometry, x: torch.Tensor, codebook: torch.Tensor, codes: torch.Tensor | None = None,
           token_offset: int = 0) -> torch.Tensor:
    """antkv_encode: x fp16 [B,Hkv,n,D] (last dim contiguous) -> codes uint8 [B,Hkv,N_cap,M]."""
    if not x.is_cuda or x.dtype != torch.float16 or x.stride(-1) != 1:
        raise ValueError("x must be an fp16 device tensor with contiguous channels")
    _need(codebook, torch.float16, "codebook")
    B, Hkv, n, _ = x.shape
    if codes is None:
        codes = torch.empty((B, Hkv, n, geom.code_bytes), dtype=torch.uint8, device=x.device)
    _need(codes, torch.uint8, "codes")
    rc = load_library().antkv_encode(geom._c, _p(x), x.stride(0), x.stride(1), x.stride(2), n, _p(codebook),
                                     _p(codes), codes.shape[2], token_offset, _stream(x))
    _check(rc, "antkv_encode")
    return codes


def topk(scores: torch.Tensor, k: int) -> torch.Tensor:
    """antkv_topk: scores fp32 [..., N] -> idx int32 [..., k]."""
    _need(scores, torch.float32, "scores")
    N = scores.shape[-1]
    rows = scores.numel() // max(N, 1)
    idx = torch.empty(scores.shape[:-1] + (k,), dtype=torch.int32, device=scores.device)
    lib = load_library()
    ws = _workspace(lib.antkv_topk_workspace(rows, N, k), scores.device)
    rc = lib.antkv_topk(_p(scores), rows, N, k, _p(idx), _p(ws), ws.numel(), _stream(scores))
    _check(rc, "antkv_topk")
    return idx


def kmeans_step(geom: Geometry, x: torch.Tensor, w: torch.Tensor, codebook: torch.Tensor):
    """antkv_kmeans_step: x fp16 [B,Hkv,n,D], w fp32 [B,Hkv,n], codebook fp16 [Hkv,M,C,d] ->
    (new codebook fp16, codes uint8 [B,Hkv,n,code_bytes], wsum fp32 [Hkv,M,C], objective fp64 [Hkv,M])."""
    _need(x, torch.float16, "x")
    _need(w, torch.float32, "w")
    _need(codebook, torch.float16, "codebook")
    B, Hkv, n, _ = x.shape
    dev = x.device
    out = torch.empty_like(codebook)
    codes = torch.empty((B, Hkv, n, geom.code_bytes), dtype=torch.uint8, device=dev)
    wsum = torch.empty((Hkv, geom.M, geom.n_centroids), dtype=torch.float32, device=dev)
    objective = torch.empty((Hkv, geom.M), dtype=torch.float64, device=dev)
    lib = load_library()
    ws = _workspace(lib.antkv_kmeans_step_workspace(geom._c), dev)
    rc = lib.antkv_kmeans_step(geom._c, _p(x), _p(w), n, _p(codebook), _p(out), _p(codes), _p(wsum),
                               _p(objective), _p(ws), ws.numel(), _stream(x))
    _check(rc, "antkv_kmeans_step")
    return out, codes, wsum, objective


def prefill_attn(geom: Geometry, q: torch.Tensor, k: torch.Tensor, v: torch.Tensor, scale: float,
                 want_stats: bool = True):
    """antkv_prefill_attn: q fp16 [B,Hq,Nq,D], k / v fp16 [B,Hkv,N,D] -> (out fp16 [B,Hq,Nq,D], row_max, row_sum)."""
    _need(q, torch.float16, "q")
    _need(k, torch.float16, "k")
    _need(v, torch.float16, "v")
    B, Hq, Nq, D = q.shape
    N = k.shape[2]
    out = torch.empty((B, Hq, Nq, D), dtype=torch.float16, device=q.device)
    row_max = torch.empty((B, Hq, Nq), dtype=torch.float32, device=q.device) if want_stats else None
    row_sum = torch.empty((B, Hq, Nq), dtype=torch.float32, device=q.device) if want_stats else None
    rc = load_library().antkv_prefill_attn(geom._c, _p(q), _p(k), _p(v), N, Nq, float(scale), _p(out),
                                           _p(row_max), _p(row_sum), _stream(q))
    _check(rc, "antkv_prefill_attn")
    return out, row_max, row_sum


def anchor_select(geom: Geometry, q: torch.Tensor, k_fp16: torch.Tensor, scale: float, k: int,
                  row_max: torch.Tensor | None = None, row_sum: torch.Tensor | None = None,
                  want_scores: bool = True):
    """antkv_anchor_select: q fp16 [B,Hq,Nq,D], k fp16 [B,Hkv,N,D] -> (idx_k, idx_v, ans_k, ans_v)."""
    _need(q, torch.float16, "q")
    _need(k_fp16, torch.float16, "k_fp16")
    B, Hkv, N, _ = k_fp16.shape
    Nq = q.shape[2]
    dev = q.device
    ans_k = torch.empty((B, Hkv, N), dtype=torch.float32, device=dev) if want_scores else None
    ans_v = torch.empty((B, Hkv, N), dtype=torch.float32, device=dev) if want_scores else None
    idx_k = torch.empty((B, Hkv, k), dtype=torch.int32, device=dev)
    idx_v = torch.empty((B, Hkv, k), dtype=torch.int32, device=dev)
    lib = load_library()
    ws = _workspace(lib.antkv_anchor_select_workspace(geom._c, N, Nq, k), dev)
    rc = lib.antkv_anchor_select(geom._c, _p(q), _p(k_fp16), N, Nq, float(scale), k, _p(row_max), _p(row_sum),
                                 _p(ans_k), _p(ans_v), _p(idx_k), _p(idx_v), _p(ws), ws.numel(), _stream(q))
    _check(rc, "antkv_anchor_select")
    return idx_k, idx_v, ans_k, ans_v


def gather_rows(geom: Geometry, x: torch.Tensor, idx: torch.Tensor, out: torch.Tensor | None = None) -> torch.Tensor:
    """antkv_gather_rows: x fp16 [B,Hkv,N,D], idx int32 [B,Hkv,k] -> rows fp16 [B,Hkv,k,D]."""
    _need(x, torch.float16, "x")
    _need(idx, torch.int32, "idx")
    B, Hkv, N, D = x.shape
    k = idx.shape[-1]
    if out is None:
        out = torch.empty((B, Hkv, k, D), dtype=torch.float16, device=x.device)
    _need(out, torch.float16, "out")
    rows = out
    rc = load_library().antkv_gather_rows(geom._c, _p(x), N, _p(idx), k, _p(rows), _stream(x))
    _check(rc, "antkv_gather_rows")
    return rows


def append_token(geom: Geometry, k_new: torch.Tensor, v_new: torch.Tensor, N: int, W: int, cb_k: torch.Tensor,
                 cb_v: torch.Tensor, codes_k: torch.Tensor, codes_v: torch.Tensor, idx_k: torch.Tensor | None,
                 rows_k: torch.Tensor | None, idx_v: torch.Tensor | None, rows_v: torch.Tensor | None) -> int:
    """antkv_append_token: retire the oldest of the W window tokens into the codes, shift the window (the last W
    entries of both anchor lists) and append the new rows at position N.  Returns the new context length N + 1."""
    _need(k_new, torch.float16, "k_new")
    _need(v_new, torch.float16, "v_new")
    _need(codes_k, torch.uint8, "codes_k")
    _need(codes_v, torch.uint8, "codes_v")
    k_k = 0 if idx_k is None else idx_k.shape[-1]
    k_v = 0 if idx_v is None else idx_v.shape[-1]
    for name, t, dt in (("idx_k", idx_k, torch.int32), ("rows_k", rows_k, torch.float16), ("idx_v", idx_v, torch.int32),
                        ("rows_v", rows_v, torch.float16)):
        if t is not None:
            _need(t, dt, name)
    rc = load_library().antkv_append_token(
        geom._c, _p(k_new), _p(v_new), N, W, _p(cb_k), _p(cb_v), _p(codes_k), _p(codes_v), codes_k.shape[2],
        _p(idx_k), _p(rows_k), k_k, _p(idx_v), _p(rows_v), k_v, _stream(k_new))
    _check(rc, "antkv_append_token")
    return N + 1


class DecodeWorkspace:
    """Caller-owned scratch for antkv_decode_attn, sized once and reused across calls."""

    def __init__(self, geom: Geometry, N: int, k_k: int, k_v: int, k_resel: int, device):
        self.nbytes = load_library().antkv_decode_attn_workspace(geom._c, N, k_k, k_v, k_resel)
        self.buf = _workspace(self.nbytes, device)


def decode_attn(geom: Geometry, q: torch.Tensor, scale: float, codes_k: torch.Tensor, codes_v: torch.Tensor,
                cb_k: torch.Tensor, cb_v: torch.Tensor, idx_k: torch.Tensor | None, rows_k: torch.Tensor | None,
                idx_v: torch.Tensor | None, rows_v: torch.Tensor | None, N: int | None = None,
                out: torch.Tensor | None = None, want_ans: bool = False, k_resel: int = 0,
                workspace: DecodeWorkspace | None = None):
    """antkv_decode_attn.  Returns out fp16 [B,Hq,D], or (out, ans_k, ans_v, resel_idx_k, resel_idx_v)."""
    _need(q, torch.float16, "q")
    _need(codes_k, torch.uint8, "codes_k")
    _need(codes_v, torch.uint8, "codes_v")
    dev = q.device
    B, Hq, D = q.shape
    Hkv = geom.Hkv
    N_cap = codes_k.shape[2]
    if N is None:
        N = N_cap
    k_k = 0 if idx_k is None else idx_k.shape[-1]
    k_v = 0 if idx_v is None else idx_v.shape[-1]
    if out is None:
        out = torch.empty((B, Hq, D), dtype=torch.float16, device=dev)
    ans_k = ans_v = rk = rv = None
    if want_ans or k_resel > 0:
        ans_k = torch.empty((B, Hkv, N), dtype=torch.float32, device=dev)
        ans_v = torch.empty((B, Hkv, N), dtype=torch.float32, device=dev)
    if k_resel > 0:
        rk = torch.empty((B, Hkv, k_resel), dtype=torch.int32, device=dev)
        rv = torch.empty((B, Hkv, k_resel), dtype=torch.int32, device=dev)
    if workspace is None:
        workspace = DecodeWorkspace(geom, N, k_k, k_v, k_resel, dev)
    rc = load_library().antkv_decode_attn(
        geom._c, _p(q), float(scale), _p(codes_k), _p(codes_v), N, N_cap, _p(cb_k), _p(cb_v),
        _p(idx_k) if k_k else None, _p(rows_k) if k_k else None, k_k,
        _p(idx_v) if k_v else None, _p(rows_v) if k_v else None, k_v,
        _p(out), _p(ans_k), _p(ans_v), _p(rk), _p(rv), k_resel, _p(workspace.buf), workspace.buf.numel(), _stream(q))
    _check(rc, "antkv_decode_attn")
    if want_ans or k_resel > 0:
        return out, ans_k, ans_v, rk, rv
    return out


def decode_attn_prerope_workspace(geom: Geometry, N: int, k_v: int, device) -> torch.Tensor:
    """A workspace of antkv_decode_attn_prerope_workspace(geom, N, k_v) bytes for decode_attn_prerope."""
    return _workspace(load_library().antkv_decode_attn_prerope_workspace(geom._c, N, k_v), device)


def decode_attn_prerope(geom: Geometry, q: torch.Tensor, scale: float, codes_k: torch.Tensor, codes_v: torch.Tensor,
                        cb_k: torch.Tensor, cb_v: torch.Tensor, idx_k: torch.Tensor | None, rows_k: torch.Tensor | None,
                        idx_v: torch.Tensor | None, rows_v: torch.Tensor | None, rope_base: float = 10000.0,
                        rope_style: int = 0, pos0: int = 0, N: int | None = None, out: torch.Tensor | None = None,
                        workspace: torch.Tensor | None = None) -> torch.Tensor:
    """antkv_decode_attn_prerope: decode attention on keys stored before RoPE.  Returns out fp16 [B,Hq,D]."""
    _need(q, torch.float16, "q")
    _need(codes_k, torch.uint8, "codes_k")
    _need(codes_v, torch.uint8, "codes_v")
    B, Hq, D = q.shape
    N_cap = codes_k.shape[2]
    if N is None:
        N = N_cap
    k_k = 0 if idx_k is None else idx_k.shape[-1]
    k_v = 0 if idx_v is None else idx_v.shape[-1]
    if out is None:
        out = torch.empty((B, Hq, D), dtype=torch.float16, device=q.device)
    if workspace is None:
        workspace = decode_attn_prerope_workspace(geom, N, k_v, q.device)
    rc = load_library().antkv_decode_attn_prerope(
        geom._c, _p(q), float(scale), _p(codes_k), _p(codes_v), N, N_cap, _p(cb_k), _p(cb_v),
        _p(idx_k) if k_k else None, _p(rows_k) if k_k else None, k_k,
        _p(idx_v) if k_v else None, _p(rows_v) if k_v else None, k_v,
        float(rope_base), int(rope_style), int(pos0), _p(out), _p(workspace), workspace.numel(), _stream(q))
    _check(rc, "antkv_decode_attn_prerope")
    return out


DECODE_FIXED_ORDER, DECODE_WIDE_TABLE = 1, 2     # ANTKV_DECODE_* of include/antkv.h


def set_decode_options(options: int) -> int:
    """antkv_set_decode_options: process-wide option mask of the one-byte-code decode kernel (DECODE_FIXED_ORDER for a
    bit-reproducible output, DECODE_WIDE_TABLE for 30-bit table entries).  Returns the previous mask."""
    return int(load_library().antkv_set_decode_options(int(options)))


STATIC_SCRATCH_BYTES = 8 << 20     # ANTKV_STATIC_SCRATCH_BYTES of include/antkv.h


def decode_attn_static(geom: Geometry, q: torch.Tensor, scale: float, codes_k: torch.Tensor, codes_v: torch.Tensor,
                       cb_k: torch.Tensor, cb_v: torch.Tensor, idx_k: torch.Tensor | None, rows_k: torch.Tensor | None,
                       idx_v: torch.Tensor | None, rows_v: torch.Tensor | None, out: torch.Tensor,
                       N: int | None = None) -> torch.Tensor:
    """antkv_decode_attn_static: decode attention with the scratch inside the library.  `out` is the caller's
    fp16 [B,Hq,D] tensor (this wrapper allocates nothing either)."""
    _need(q, torch.float16, "q")
    _need(codes_k, torch.uint8, "codes_k")
    _need(codes_v, torch.uint8, "codes_v")
    _need(out, torch.float16, "out")
    N_cap = codes_k.shape[2]
    if N is None:
        N = N_cap
    k_k = 0 if idx_k is None else idx_k.shape[-1]
    k_v = 0 if idx_v is None else idx_v.shape[-1]
    rc = load_library().antkv_decode_attn_static(
        geom._c, _p(q), float(scale), _p(codes_k), _p(codes_v), N, N_cap, _p(cb_k), _p(cb_v),
        _p(idx_k) if k_k else None, _p(rows_k) if k_k else None, k_k,
        _p(idx_v) if k_v else None, _p(rows_v) if k_v else None, k_v, _p(out), _stream(q))
    _check(rc, "antkv_decode_attn_static")
    return out
