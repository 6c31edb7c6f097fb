"""Binding of libadamas.so: argument marshalling only, through ctypes, and for the calls of a decoding loop in native
code (csrc/marshal.cpp), which hands back what it does not take as it is.

Every function mirrors the C entry point of the same name in include/adamas.h, takes torch
tensors that already live on the GPU, checks dtype / device / contiguity, and passes raw
device pointers plus the current HIP stream.  All arithmetic happens in the HIP kernels; there
is no CPU or PyTorch fallback: if the shared library is missing and cannot be built, loading
raises.
"""

from __future__ import annotations

import ctypes
import os
from typing import Optional, Sequence

from . import build as _build

EXPORTED_SYMBOLS = (
    "adamas_status_string",
    "adamas_build_id",
    "adamas_last_hip_error",
    "adamas_workspace_bytes",
    "adamas_encode_keys",
    "adamas_encode_query",
    "adamas_manhattan_distance",
    "adamas_select_topk",
    "adamas_sparse_attn",
    "adamas_decode_step",
    "adamas_decode_step_stages",
    "adamas_decode_step_static",
    "adamas_phase_trace",
    "adamas_stream_read",
    "adamas_decode_step_paged",
    "adamas_full_attn_workspace_bytes",
    "adamas_full_attn",
)

HEAD_DIM = 128
CODE_ROW_BYTES = 32
VARIANT_NO_HADAMARD = 1
VARIANT_L2 = 2
STAGE_SCAN, STAGE_SELECT_ATTN, STAGE_ALL = 1, 2, 3
STATIC_SCRATCH_BYTES = 16 << 20


class AdamasError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        hip = library().adamas_last_hip_error() if status == -4 else 0
        super().__init__("%s: %s (%d)%s" % (where, adamas_status_string(status), status,
                                            " hipError %d" % hip if hip else ""))


class Config(ctypes.Structure):
    """Mirror of struct adamas_config."""
    _fields_ = [
        ("head_dim", ctypes.c_int32),
        ("num_q_heads", ctypes.c_int32),
        ("num_kv_heads", ctypes.c_int32),
        ("variant", ctypes.c_uint32),
        ("pool_tokens", ctypes.c_int64),
        ("thr_k", ctypes.c_float * 7),
        ("thr_q", ctypes.c_float * 7),
        ("sm_scale", ctypes.c_float),
        ("code_bits", ctypes.c_int32),
    ]

    @property
    def code_row_bytes(self) -> int:
        return self.head_dim // 8 * (self.code_bits or 2)

    @classmethod
    def make(cls, num_q_heads: int, num_kv_heads: int, pool_tokens: int,
             thr_k: Sequence[float] = (-1.0, 0.0, 1.0), thr_q: Optional[Sequence[float]] = None,
             sm_scale: float = 0.0, head_dim: int = HEAD_DIM, variant: int = 0,
             code_bits: int = 0) -> "Config":
        """thr_k / thr_q hold 2^code_bits - 1 thresholds (three for the default 2-bit codes)."""
        thr_q = thr_k if thr_q is None else thr_q
        n_thr = (1 << (code_bits or 2)) - 1
        if len(thr_k) != n_thr or len(thr_q) != n_thr:
            raise ValueError("%d thresholds needed for %d-bit codes" % (n_thr, code_bits or 2))
        pad = lambda t: (ctypes.c_float * 7)(*(list(t) + [0.0] * (7 - len(t))))
        return cls(head_dim, num_q_heads, num_kv_heads, variant, pool_tokens, pad(thr_k), pad(thr_q),
                   sm_scale, code_bits)


_lib = None
_marshal = None  # the native marshalling module, once the library is loaded; None: ctypes only
torch = None    # the module, once the library is loaded (imported there, not with this package)


def library_path():
    return _build.LIB


def library() -> ctypes.CDLL:
    """Loads libadamas.so, building it first (in a child process, before anything here touches
    the GPU library) when it is missing or was built from sources other than the tree's.  The
    environment variable ADAMAS_LIBRARY names another built library to load instead."""
    global _lib, _marshal, torch
    if _lib is None:
        # torch first: the process then has one HIP runtime (the one torch ships), and this
        # library, which only needs the public HIP launch API, binds to it.
        import torch as torch_module
        path = os.environ.get("ADAMAS_LIBRARY")     # a library built elsewhere: loaded as it is
        if not path:
            if _build.is_stale():
                _build.build()
            path = str(_build.LIB)
        lib = ctypes.CDLL(path)
        vp, i32, i64, sz = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64, ctypes.c_size_t
        cfgp = ctypes.POINTER(Config)
        lib.adamas_status_string.restype = ctypes.c_char_p
        lib.adamas_status_string.argtypes = [ctypes.c_int]
        lib.adamas_build_id.restype = ctypes.c_char_p
        lib.adamas_build_id.argtypes = []
        lib.adamas_last_hip_error.restype = ctypes.c_int
        lib.adamas_last_hip_error.argtypes = []
        lib.adamas_workspace_bytes.restype = sz
        lib.adamas_workspace_bytes.argtypes = [cfgp, i32, i64, i32]
        lib.adamas_encode_keys.restype = ctypes.c_int
        lib.adamas_encode_keys.argtypes = [cfgp, vp, vp, i64, i64, vp]
        lib.adamas_encode_query.restype = ctypes.c_int
        lib.adamas_encode_query.argtypes = [cfgp, vp, vp, i32, vp]
        lib.adamas_manhattan_distance.restype = ctypes.c_int
        lib.adamas_manhattan_distance.argtypes = [cfgp, vp, vp, vp, vp, i32, vp, i64, vp]
        lib.adamas_select_topk.restype = ctypes.c_int
        lib.adamas_select_topk.argtypes = [cfgp, vp, vp, vp, vp, i32, i32, vp, vp, i64, vp, sz, vp]
        lib.adamas_sparse_attn.restype = ctypes.c_int
        lib.adamas_sparse_attn.argtypes = [cfgp, vp, vp, vp, vp, vp, i32, i32, vp, i64, vp, sz, vp]
        lib.adamas_decode_step.restype = ctypes.c_int
        lib.adamas_decode_step.argtypes = [cfgp, vp, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp,
                                           i64, vp, sz, vp]
        lib.adamas_decode_step_static.restype = ctypes.c_int
        lib.adamas_decode_step_static.argtypes = [cfgp, vp, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp,
                                                  vp, i64, vp]
        lib.adamas_phase_trace.restype = ctypes.c_int
        lib.adamas_phase_trace.argtypes = [vp, vp, i64]
        lib.adamas_decode_step_paged.restype = ctypes.c_int
        lib.adamas_decode_step_paged.argtypes = [cfgp, vp, vp, vp, vp, vp, vp, vp, i32, i32, vp,
                                                 i32, i32, vp, vp, i64, vp, sz, vp,
                                                 ctypes.c_uint32]
        lib.adamas_full_attn_workspace_bytes.restype = sz
        lib.adamas_full_attn_workspace_bytes.argtypes = [cfgp, i32, i64]
        lib.adamas_full_attn.restype = ctypes.c_int
        lib.adamas_full_attn.argtypes = [cfgp, vp, vp, vp, vp, vp, i32, vp, i64, vp, sz, vp]
        lib.adamas_stream_read.restype = ctypes.c_int
        lib.adamas_stream_read.argtypes = [vp, sz, vp, vp]
        lib.adamas_decode_step_stages.restype = ctypes.c_int
        lib.adamas_decode_step_stages.argtypes = lib.adamas_decode_step.argtypes + [ctypes.c_uint32]
        torch = torch_module
        _marshal = _load_marshal(lib)
        _lib = lib
    return _lib


def _load_marshal(lib):
    """The native marshalling module, bound to this library's entry points; built if it is missing or was built from
    other sources.  None, with a warning, where it cannot be built or torch has no GPU support to ask for a stream: every
    call then goes through ctypes."""
    import importlib.machinery
    import importlib.util
    import subprocess
    import warnings

    def load():
        loader = importlib.machinery.ExtensionFileLoader("_marshal", str(_build.MARSHAL_LIB))
        module = importlib.util.module_from_spec(importlib.util.spec_from_loader("_marshal", loader))
        loader.exec_module(module)
        return module

    try:
        # (a module that has been loaded once stays what it is in this process: look before loading)
        if not _build.MARSHAL_LIB.exists() or _build.marshal_id().encode() not in _build.MARSHAL_LIB.read_bytes():
            _build.build_marshal()
        module = load()
        import torch as torch_module
        address = lambda fn: ctypes.cast(fn, ctypes.c_void_p).value
        module.bind(Config, torch_module._C._cuda_getDevice, torch_module._C._cuda_getCurrentRawStream,
                    address(lib.adamas_decode_step), address(lib.adamas_decode_step_paged),
                    address(lib.adamas_encode_keys), address(lib.adamas_full_attn))
    except (ImportError, OSError, AttributeError, subprocess.CalledProcessError) as e:
        warnings.warn("no native argument marshalling (%s: %s): calls go through ctypes, some microseconds slower each"
                      % (type(e).__name__, e), RuntimeWarning, stacklevel=3)
        return None
    return module


def adamas_status_string(status: int) -> str:
    return library().adamas_status_string(int(status)).decode()


def build_id() -> str:
    """Hash of the sources the loaded library was built from."""
    return library().adamas_build_id().decode()


def adamas_workspace_bytes(cfg: Config, batch: int, max_seq_len: int, k: int) -> int:
    return int(library().adamas_workspace_bytes(ctypes.byref(cfg), batch, max_seq_len, k))


# ------------------------------------------------------------------ tensor marshalling

# A call of the library from Python is bound by what happens here (a decode step on a small cache: 20 us a
# call, of which 9 on the GPU), so the modules and shapes are looked at once: shapes are compared as they are, the
# current stream is asked for without building a Stream object.

def _ptr(t, dtype, name, shape=None, optional=False):
    if t is None:
        if optional:
            return None
        raise TypeError("%s must not be None" % name)
    if not isinstance(t, torch.Tensor):
        raise TypeError("%s must be a torch.Tensor" % name)
    if not t.is_cuda:
        raise ValueError("%s must live on the GPU" % name)
    if t.dtype != dtype:
        raise ValueError("%s must have dtype %s, got %s" % (name, dtype, t.dtype))
    if not t.is_contiguous():
        raise ValueError("%s must be contiguous" % name)
    if shape is not None and t.shape != shape:      # a torch.Size is a tuple
        raise ValueError("%s must have shape %s, got %s" % (name, tuple(shape), tuple(t.shape)))
    return t.data_ptr()


def _stream(stream):
    if stream is None:
        return torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice())
    return stream.cuda_stream if hasattr(stream, "cuda_stream") else int(stream)


def _check(rc, where):
    if rc != 0:
        raise AdamasError(rc, where)


# The functions with a native form try that first; it returns a status, or None for arguments that it does not take as they
# are, and the checks below then say what is wrong with them (or accept them).

def adamas_encode_keys(cfg: Config, K, codes, row_begin: int, n_rows: int, stream=None) -> None:
    if _marshal is not None:
        rc = _marshal.encode_keys(cfg, K, codes, row_begin, n_rows, None if stream is None else _stream(stream))
        if rc is not None:
            return _check(rc, "adamas_encode_keys")
    lib = _lib or library()
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    rc = lib.adamas_encode_keys(
        ctypes.byref(cfg), _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(codes, torch.uint8, "codes", (hkv, pool, cfg.code_row_bytes)), row_begin, n_rows,
        _stream(stream))
    _check(rc, "adamas_encode_keys")


def adamas_encode_query(cfg: Config, q, qcodes, stream=None) -> None:
    lib = _lib or library()
    batch = q.shape[0]
    rc = lib.adamas_encode_query(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(qcodes, torch.uint8, "qcodes", (batch, cfg.num_q_heads, cfg.code_row_bytes)), batch,
        _stream(stream))
    _check(rc, "adamas_encode_query")


def adamas_decode_step_paged(cfg: Config, q, K, V, codes, page_table, page_tokens: int, seq_len,
                             k: int, out, max_seq_len: int, workspace, k_new=None, v_new=None,
                             idx_out=None, stream=None, stages=STAGE_ALL) -> None:
    if _marshal is not None:
        rc = _marshal.decode_step_paged(cfg, q, K, V, codes, page_table, page_tokens, seq_len, k, out, max_seq_len, workspace,
                                        k_new, v_new, idx_out, None if stream is None else _stream(stream), stages)
        if rc is not None:
            return _check(rc, "adamas_decode_step_paged")
    lib = _lib or library()
    batch = q.shape[0]
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    if page_table.dim() != 2 or page_table.shape[0] != batch:
        raise ValueError("page_table must have shape (batch, max_pages)")
    rc = lib.adamas_decode_step_paged(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(k_new, torch.bfloat16, "k_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(v_new, torch.bfloat16, "v_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(V, torch.bfloat16, "V", (hkv, pool, cfg.head_dim)),
        _ptr(codes, torch.uint8, "codes", (hkv, pool, cfg.code_row_bytes)),
        _ptr(page_table, torch.int32, "page_table"), page_table.shape[1], int(page_tokens),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch, k,
        _ptr(out, torch.float32, "out", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(idx_out, torch.int32, "idx_out", (batch, cfg.num_q_heads, k), optional=True),
        max_seq_len, _ptr(workspace, torch.uint8, "workspace"), workspace.numel(), _stream(stream),
        int(stages))
    _check(rc, "adamas_decode_step_paged")


def adamas_full_attn_workspace_bytes(cfg: Config, batch: int, max_seq_len: int) -> int:
    return int(library().adamas_full_attn_workspace_bytes(ctypes.byref(cfg), batch, max_seq_len))


def adamas_full_attn(cfg: Config, q, K, V, seq_start, seq_len, out, max_seq_len: int, workspace,
                     stream=None) -> None:
    if _marshal is not None:
        rc = _marshal.full_attn(cfg, q, K, V, seq_start, seq_len, out, max_seq_len, workspace,
                                None if stream is None else _stream(stream))
        if rc is not None:
            return _check(rc, "adamas_full_attn")
    lib = _lib or library()
    batch = q.shape[0]
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    rc = lib.adamas_full_attn(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(V, torch.bfloat16, "V", (hkv, pool, cfg.head_dim)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch,
        _ptr(out, torch.float32, "out", (batch, cfg.num_q_heads, cfg.head_dim)),
        max_seq_len, _ptr(workspace, torch.uint8, "workspace"), workspace.numel(), _stream(stream))
    _check(rc, "adamas_full_attn")


def adamas_stream_read(src, sink, stream=None) -> None:
    """Reads every byte of the uint8 tensor `src` once (measurement aid); `sink` int32, >= 1 element."""
    lib = _lib or library()
    rc = lib.adamas_stream_read(_ptr(src, torch.uint8, "src"), src.numel(),
                                      _ptr(sink, torch.int32, "sink"), _stream(stream))
    _check(rc, "adamas_stream_read")


def adamas_manhattan_distance(cfg: Config, qcodes, codes, seq_start, seq_len, dist_out,
                              stream=None) -> None:
    lib = _lib or library()
    batch = qcodes.shape[0]
    max_seq_len = dist_out.shape[2]
    rc = lib.adamas_manhattan_distance(
        ctypes.byref(cfg),
        _ptr(qcodes, torch.uint8, "qcodes", (batch, cfg.num_q_heads, cfg.code_row_bytes)),
        _ptr(codes, torch.uint8, "codes", (cfg.num_kv_heads, cfg.pool_tokens, cfg.code_row_bytes)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch,
        _ptr(dist_out, torch.uint16, "dist_out", (batch, cfg.num_q_heads, max_seq_len)),
        max_seq_len, _stream(stream))
    _check(rc, "adamas_manhattan_distance")


def adamas_select_topk(cfg: Config, qcodes, codes, seq_start, seq_len, k: int, idx_out,
                       max_seq_len: int, workspace, dist_out=None, stream=None) -> None:
    lib = _lib or library()
    batch = qcodes.shape[0]
    rc = lib.adamas_select_topk(
        ctypes.byref(cfg),
        _ptr(qcodes, torch.uint8, "qcodes", (batch, cfg.num_q_heads, cfg.code_row_bytes)),
        _ptr(codes, torch.uint8, "codes", (cfg.num_kv_heads, cfg.pool_tokens, cfg.code_row_bytes)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch, k,
        _ptr(idx_out, torch.int32, "idx_out", (batch, cfg.num_q_heads, k)),
        _ptr(dist_out, torch.uint16, "dist_out", (batch, cfg.num_q_heads, max_seq_len),
             optional=True),
        max_seq_len, _ptr(workspace, torch.uint8, "workspace"), workspace.numel(),
        _stream(stream))
    _check(rc, "adamas_select_topk")


def adamas_sparse_attn(cfg: Config, q, K, V, seq_start, idx, out, max_seq_len: int, workspace,
                       stream=None) -> None:
    lib = _lib or library()
    batch, _, k = idx.shape
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    rc = lib.adamas_sparse_attn(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(V, torch.bfloat16, "V", (hkv, pool, cfg.head_dim)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(idx, torch.int32, "idx", (batch, cfg.num_q_heads, k)), batch, k,
        _ptr(out, torch.float32, "out", (batch, cfg.num_q_heads, cfg.head_dim)), max_seq_len,
        _ptr(workspace, torch.uint8, "workspace"), workspace.numel(), _stream(stream))
    _check(rc, "adamas_sparse_attn")




def adamas_decode_step(cfg: Config, q, K, V, codes, seq_start, seq_len, k: int, out,
                       max_seq_len: int, workspace, k_new=None, v_new=None, idx_out=None,
                       stream=None) -> None:
    if _marshal is not None:
        rc = _marshal.decode_step(cfg, q, K, V, codes, seq_start, seq_len, k, out, max_seq_len, workspace, k_new, v_new, idx_out,
                                  None if stream is None else _stream(stream))
        if rc is not None:
            return _check(rc, "adamas_decode_step")
    adamas_decode_step_stages(cfg, q, K, V, codes, seq_start, seq_len, k, out, max_seq_len,
                              workspace, k_new=k_new, v_new=v_new, idx_out=idx_out, stream=stream,
                              stages=None)


TRACE_SLOTS = 16


def adamas_phase_trace(scan_records, select_records) -> None:
    """Profiling builds only: int64 tensors [n_records, TRACE_SLOTS] on the GPU that receive the
    kernels' phase stamps (None, None switches them off)."""
    lib = _lib or library()
    n = 0
    for t in (scan_records, select_records):
        if t is not None:
            if t.dim() != 2 or t.shape[1] != TRACE_SLOTS:
                raise ValueError("trace buffers must have shape (n_records, %d)" % TRACE_SLOTS)
            n = t.shape[0] if n == 0 else n
            if t.shape[0] != n:
                raise ValueError("both trace buffers must hold the same number of records")
    rc = lib.adamas_phase_trace(_ptr(scan_records, torch.int64, "scan_records", optional=True),
                                      _ptr(select_records, torch.int64, "select_records",
                                           optional=True), n)
    _check(rc, "adamas_phase_trace")


def adamas_decode_step_static(cfg: Config, q, K, V, codes, seq_start, seq_len, k: int, out,
                              max_seq_len: int, k_new=None, v_new=None, idx_out=None,
                              stream=None) -> None:
    """adamas_decode_step on the library's own static scratch array: no workspace argument."""
    lib = _lib or library()
    batch = q.shape[0]
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    rc = lib.adamas_decode_step_static(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(k_new, torch.bfloat16, "k_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(v_new, torch.bfloat16, "v_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(V, torch.bfloat16, "V", (hkv, pool, cfg.head_dim)),
        _ptr(codes, torch.uint8, "codes", (hkv, pool, cfg.code_row_bytes)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch, k,
        _ptr(out, torch.float32, "out", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(idx_out, torch.int32, "idx_out", (batch, cfg.num_q_heads, k), optional=True),
        max_seq_len, _stream(stream))
    _check(rc, "adamas_decode_step_static")


def adamas_decode_step_stages(cfg: Config, q, K, V, codes, seq_start, seq_len, k: int, out,
                              max_seq_len: int, workspace, k_new=None, v_new=None, idx_out=None,
                              stream=None, stages=STAGE_ALL) -> None:
    """stages=None calls the plain adamas_decode_step entry point."""
    lib = _lib or library()
    batch = q.shape[0]
    hkv, pool = cfg.num_kv_heads, cfg.pool_tokens
    fn = lib.adamas_decode_step if stages is None else lib.adamas_decode_step_stages
    extra = () if stages is None else (int(stages),)
    rc = fn(
        ctypes.byref(cfg), _ptr(q, torch.bfloat16, "q", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(k_new, torch.bfloat16, "k_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(v_new, torch.bfloat16, "v_new", (batch, hkv, cfg.head_dim), optional=True),
        _ptr(K, torch.bfloat16, "K", (hkv, pool, cfg.head_dim)),
        _ptr(V, torch.bfloat16, "V", (hkv, pool, cfg.head_dim)),
        _ptr(codes, torch.uint8, "codes", (hkv, pool, cfg.code_row_bytes)),
        _ptr(seq_start, torch.int64, "seq_start", (batch,)),
        _ptr(seq_len, torch.int32, "seq_len", (batch,)), batch, k,
        _ptr(out, torch.float32, "out", (batch, cfg.num_q_heads, cfg.head_dim)),
        _ptr(idx_out, torch.int32, "idx_out", (batch, cfg.num_q_heads, k), optional=True),
        max_seq_len, _ptr(workspace, torch.uint8, "workspace"), workspace.numel(),
        _stream(stream), *extra)
    _check(rc, "adamas_decode_step")
