"""Binding of include/seco.h: argument marshalling only.

Tensor arguments are torch tensors on the GPU, laid out [batch, head, row, head_dim] with a
contiguous last dimension (any outer strides).  The calls that take tensors go through a small
extension module (csrc/binding_ext.cpp), which builds the `seco_desc`, allocates what the caller
did not supply, passes raw device pointers and the current HIP stream, and raises SecoError on a
non-zero status; host-only calls (selection, weights, sizes, profiler) go through ctypes.
"""
from __future__ import annotations

import ctypes as C
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
# SECO_LIBRARY overrides the path (e.g. to try a library built with other tile parameters)
_LIB_PATH = os.environ.get("SECO_LIBRARY") or os.path.join(_HERE, "libseco_hip.so")
_lib = None
_ext = None

SECO_F32, SECO_BF16 = 0, 1
SECO_OP_FWD, SECO_OP_BWD = 0, 1


class SecoDesc(C.Structure):
    _fields_ = [
        ("batch", C.c_int32), ("n_q_heads", C.c_int32), ("n_kv_heads", C.c_int32), ("head_dim", C.c_int32),
        ("chunk_len", C.c_int32), ("q_start", C.c_int32), ("dtype", C.c_int32), ("softmax_scale", C.c_float),
        ("q_stride", C.c_int64 * 3), ("o_stride", C.c_int64 * 3),
        ("kv_stride", C.c_int64 * 3), ("g_stride", C.c_int64 * 3),
    ]


class SecoError(RuntimeError):
    def __init__(self, status, where):
        self.status = status
        super().__init__(f"{where}: {seco_strerror(status)} (status {status})")


def library_path():
    return _LIB_PATH


def load_library():
    """Load libseco_hip.so (built by paper_2505_16710_amd.build); raises if it is missing."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} not found: run `python -m paper_2505_16710_amd.build` "
                          "(there is no fallback path)")
    lib = C.CDLL(_LIB_PATH)
    vp, fp, i32, i64, sz = C.c_void_p, C.c_void_p, C.c_int32, C.c_int64, C.c_size_t
    dp = C.POINTER(SecoDesc)
    lib.seco_chunk_attn_fwd.argtypes = [dp, vp, vp, vp, vp, fp, vp, sz, vp]
    lib.seco_chunk_attn_bwd.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp, vp, sz, vp]
    lib.spaco_chunk_attn_bwd.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp,
                                         C.POINTER(C.c_float), i32, i32, vp, sz, vp]
    lib.spaco_chunk_attn_bwd_sparse_dq.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp, C.POINTER(C.c_float),
                                                   C.POINTER(C.c_float), i32, i32, vp, sz, vp]
    lib.spaco_chunk_attn_bwd_sparse_dq.restype = C.c_int
    lib.seco_chunk_attn_bwd_noalloc.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp, vp]
    lib.seco_chunk_attn_bwd_noalloc.restype = C.c_int
    lib.seco_chunk_attn_bwd_gather.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32, vp, sz, vp]
    lib.seco_chunk_attn_bwd_gather.restype = C.c_int
    lib.spaco_chunk_attn_bwd_gather.argtypes = [dp, vp, vp, vp, vp, fp, vp, vp, fp, fp, fp, i64, i32,
                                                C.POINTER(C.c_float), i32, i32, vp, sz, vp]
    lib.spaco_chunk_attn_bwd_gather.restype = C.c_int
    lib.kvgrad_zero.argtypes = [dp, fp, fp, i64, i64, vp]
    lib.kvgrad_accumulate.argtypes = [dp, fp, fp, fp, fp, C.c_float, i64, i64, vp]
    lib.kv_append.argtypes = [dp, vp, vp, vp, vp, vp]
    lib.kvgrad_readout.argtypes = [dp, fp, fp, vp, vp, C.c_float, vp]
    lib.kv_append.restype = lib.kvgrad_readout.restype = C.c_int
    lib.kv_append_rope.argtypes = [dp, vp, vp, vp, vp, C.c_float, vp]
    lib.kvgrad_readout_rope.argtypes = [dp, fp, fp, vp, vp, C.c_float, C.c_float, vp]
    lib.rope_rotate.argtypes = [dp, i32, vp, vp, i64, C.c_float, i32, vp]
    lib.kv_append_rope.restype = lib.kvgrad_readout_rope.restype = lib.rope_rotate.restype = C.c_int
    lib.spaco_select_chunks.argtypes = [C.c_uint64, C.c_uint64, i32, i32, C.POINTER(i32)]
    lib.spaco_chunk_weights.argtypes = [C.POINTER(i32), i32, i32, C.c_float, C.POINTER(C.c_float)]
    lib.spaco_gather_row_weights.argtypes = [C.POINTER(i32), i32, i32, i32, C.c_float, C.POINTER(C.c_float)]
    lib.spaco_gather_row_weights.restype = C.c_int
    lib.spaco_percall_weights.argtypes = [C.c_uint64, C.c_uint64, i32, i32, C.POINTER(C.c_float)]
    lib.spaco_percall_weights.restype = C.c_int
    lib.spaco_select_bernoulli.argtypes = [C.c_uint64, C.c_uint64, i32, C.c_double, C.POINTER(i32), C.POINTER(i32)]
    lib.spaco_select_bernoulli.restype = C.c_int
    lib.spaco_compensation_factor.argtypes = [i32, i32, C.c_float]
    lib.spaco_compensation_factor.restype = C.c_float
    lib.seco_workspace_bytes.argtypes = [dp, C.c_int]
    lib.seco_launch_plan.argtypes = [dp, i32, C.POINTER(i32)]
    lib.seco_launch_plan.restype = C.c_int
    lib.seco_device_info.argtypes = [C.POINTER(i32), C.POINTER(i32)]
    lib.seco_device_info.restype = C.c_int
    lib.seco_workspace_bytes.restype = sz
    lib.seco_strerror.argtypes = [C.c_int]
    lib.seco_strerror.restype = C.c_char_p
    lib.seco_profile_enable.argtypes = [C.c_int]
    lib.seco_profile_read.argtypes = [C.POINTER(C.c_double), C.POINTER(C.c_int64)]
    lib.seco_profile_enable_kinds.argtypes = [C.c_uint32]
    lib.seco_profile_set_kinds.argtypes = [C.c_uint32]
    lib.seco_profile_set_kinds.restype = C.c_int
    lib.seco_profile_enable.restype = lib.seco_profile_read.restype = lib.seco_profile_enable_kinds.restype = C.c_int
    for name in ("seco_chunk_attn_fwd", "seco_chunk_attn_bwd", "spaco_chunk_attn_bwd", "kvgrad_zero",
                 "kvgrad_accumulate", "spaco_select_chunks", "spaco_chunk_weights"):
        getattr(lib, name).restype = C.c_int
    _lib = lib
    return lib


def _load_ext():
    """The extension module, bound to the library's entry points; raises if either has not been built."""
    global _ext
    import torch  # noqa: F401  (the extension links against its libraries)
    load_library()
    try:
        from . import _seco_ext
    except ImportError as e:
        raise ImportError(f"{e}: run `python -m paper_2505_16710_amd.build` (there is no fallback path)") from e
    _seco_ext.init(_LIB_PATH, SecoError)
    _ext = _seco_ext
    return _ext


def seco_strerror(status):
    return load_library().seco_strerror(int(status)).decode()


def _check(status, where):
    if status != 0:
        raise SecoError(status, where)


def _dtype_code(t):
    import torch
    if t.dtype == torch.bfloat16:
        return SECO_BF16
    if t.dtype == torch.float32:
        return SECO_F32
    raise TypeError(f"unsupported dtype {t.dtype}")


def _strides3(t):
    if t.dim() != 4 or t.stride(3) != 1:
        raise ValueError("expected a [batch, head, row, head_dim] tensor with contiguous head_dim")
    return (C.c_int64 * 3)(t.stride(0), t.stride(1), t.stride(2))


def make_desc(q, k_cache, q_start, scale, o=None, g=None):
    """seco_desc for a chunk call; o defaults to q's strides, g to a contiguous fp32 cache."""
    B, Hq, Cn, D = q.shape
    d = SecoDesc()
    d.batch, d.n_q_heads, d.n_kv_heads, d.head_dim = B, Hq, k_cache.shape[1], D
    d.chunk_len, d.q_start, d.dtype, d.softmax_scale = Cn, int(q_start), _dtype_code(q), float(scale)
    d.q_stride = _strides3(q)
    d.o_stride = _strides3(o if o is not None else q)
    d.kv_stride = _strides3(k_cache)
    d.g_stride = _strides3(g) if g is not None else _strides3(k_cache)
    return d


def seco_workspace_bytes(desc, op):
    n = load_library().seco_workspace_bytes(C.byref(desc), int(op))
    if n == C.c_size_t(-1).value:
        raise SecoError(-2, "seco_workspace_bytes")
    return n


def seco_chunk_attn_fwd(q, k_cache, v_cache, q_start, scale, o=None, lse=None, stream=None, ws=None):
    """O, LSE of one chunk against cache rows [0, q_start + C).  Returns (o, lse).

    ws: optional uint8 workspace tensor (see seco_workspace_bytes); allocated here when the shape wants one,
    False to pass none."""
    return (_ext or _load_ext()).fwd(q, k_cache, v_cache, q_start, scale, o, lse, stream, ws)


def seco_chunk_attn_bwd(q, k_cache, v_cache, o, lse, d_o, gk, gv, q_start, scale, d_q=None, ws=None, stream=None):
    """dQ of the chunk; adds the chunk's dK/dV into gk, gv (fp32, whole cache).  Returns d_q."""
    return (_ext or _load_ext()).bwd(q, k_cache, v_cache, o, lse, d_o, gk, gv, q_start, scale, d_q, ws, stream, None, None,
                                     None)


STATIC_SCRATCH_BYTES = 40 << 20


def seco_chunk_attn_bwd_noalloc(q, k_cache, v_cache, o, lse, d_o, d_q, gk, gv, q_start, scale, stream=None):
    """seco_chunk_attn_bwd on the library's own static device scratch: no workspace argument, nothing allocated here
    or in the library (d_q must be supplied).  Returns d_q."""
    return (_ext or _load_ext()).bwd_noalloc(q, k_cache, v_cache, o, lse, d_o, d_q, gk, gv, q_start, scale, stream)


def spaco_chunk_attn_bwd(q, k_cache, v_cache, o, lse, d_o, gk, gv, q_start, scale, chunk_weight, weight_chunk_len,
                         d_q=None, ws=None, stream=None, dq_weight=None):
    """As seco_chunk_attn_bwd with per-chunk weights (host sequence of floats) on the dK/dV contributions.
    With dq_weight (one non-negative float per chunk) the call is spaco_chunk_attn_bwd_sparse_dq: dQ visits only
    the chunks with a non-zero dq weight and scales their terms by it."""
    if chunk_weight is None:
        raise TypeError("chunk_weight must be a sequence of floats")
    return (_ext or _load_ext()).bwd(q, k_cache, v_cache, o, lse, d_o, gk, gv, q_start, scale, d_q, ws, stream, chunk_weight,
                                     weight_chunk_len, dq_weight)


def seco_chunk_attn_bwd_gather(q_rows, k_cache, v_cache, o, lse, d_o_rows, gk, gv, q_start, scale, chunk_len,
                               row_stats, d_q=None, ws=None, stream=None, row_weight=None, weight_chunk_len=None):
    """Backward of one chunk in the transposed order: dQ of the chunk's first `chunk_len` rows of q_rows, and the
    chunk's own gK/gV rows from all of q_rows / d_o_rows (the chunk's rows followed by every later row).
    row_stats: fp32 [2, B, Hq, stat_rows] kept by the caller over the whole backward pass.
    row_weight (host floats, one per chunk of weight_chunk_len rows counted from the call's first row; default
    chunk_len): the call is spaco_chunk_attn_bwd_gather."""
    return (_ext or _load_ext()).bwd_gather(q_rows, k_cache, v_cache, o, lse, d_o_rows, gk, gv, q_start, scale, chunk_len,
                                            row_stats, d_q, ws, stream, row_weight, weight_chunk_len)


def kvgrad_zero(gk, gv, row_begin=0, row_end=None, stream=None):
    """Zero rows [row_begin, row_end) of the fp32 KV-gradient buffers (either may be None)."""
    (_ext or _load_ext()).zero(gk, gv, row_begin, row_end, stream)


def kvgrad_accumulate(dst_k, dst_v, src_k, src_v, scale, row_begin=0, row_end=None, stream=None):
    """dst[rows] += scale * src[rows] on fp32 KV-gradient buffers with identical strides."""
    (_ext or _load_ext()).accumulate(dst_k, dst_v, src_k, src_v, scale, row_begin, row_end, stream)


def kv_append(k_new, v_new, k_cache, v_cache, row_begin, stream=None, rope_base=None):
    """Write the chunk's keys / values ([B, Hkv, C, D]) into cache rows [row_begin, row_begin + C); with rope_base the
    keys are rotated for their positions on the way (kv_append_rope)."""
    (_ext or _load_ext()).append(k_new, v_new, k_cache, v_cache, row_begin, stream, rope_base)


def kvgrad_readout(gk, gv, row_begin, n_rows, dtype, scaler=1.0, d_k=None, d_v=None, stream=None, rope_base=None):
    """(d_k, d_v) = scaler * (gk, gv)[rows row_begin .. row_begin + n_rows) in the storage dtype; with rope_base the
    key part is turned back by the rows' rotary angles (kvgrad_readout_rope)."""
    return (_ext or _load_ext()).readout(gk, gv, row_begin, n_rows, dtype, scaler, d_k, d_v, stream, rope_base)


def rope_rotate(x, pos_start, rope_base, inverse=False, out=None, stream=None):
    """Rotary position embedding of x [B, H, C, D] (row r at position pos_start + r), or its inverse / transpose."""
    return (_ext or _load_ext()).rotate(x, pos_start, rope_base, inverse, out, stream)


def spaco_select_chunks(seed, step, k, t):
    """t distinct chunk indices of 0..k-1, descending (list of int)."""
    out = (C.c_int32 * max(int(t), 1))()
    _check(load_library().spaco_select_chunks(int(seed), int(step), int(k), int(t), out), "spaco_select_chunks")
    return list(out[:t])


def spaco_percall_weights(seed, step, j, t):
    """Weight vector w[0..j] of call j when every call draws min(t, j) of its earlier chunks itself (list of float)."""
    w = (C.c_float * (int(j) + 1))()
    _check(load_library().spaco_percall_weights(int(seed), int(step), int(j), int(t), w), "spaco_percall_weights")
    return list(w)


def spaco_select_bernoulli(seed, step, k, q):
    """Every chunk of 0..k-1 selected independently with probability q; indices descending (list of int)."""
    out = (C.c_int32 * max(int(k), 1))()
    n = C.c_int32(0)
    _check(load_library().spaco_select_bernoulli(int(seed), int(step), int(k), float(q), out, C.byref(n)),
           "spaco_select_bernoulli")
    return list(out[:n.value])


def spaco_compensation_factor(k, t, cap=0.0):
    """k/t, limited to cap when cap > 0."""
    lam = load_library().spaco_compensation_factor(int(k), int(t), float(cap))
    if lam < 0:
        raise SecoError(-8, "spaco_compensation_factor")
    return lam


def spaco_chunk_weights(selected, j, factor):
    """Weight vector w[0..j] of the backward call for chunk j (list of float)."""
    sel = (C.c_int32 * max(len(selected), 1))(*[int(i) for i in selected])
    w = (C.c_float * (int(j) + 1))()
    _check(load_library().spaco_chunk_weights(sel, len(selected), int(j), float(factor), w), "spaco_chunk_weights")
    return list(w)


def spaco_gather_row_weights(selected, i, k, factor):
    """Row weights w[0 .. k-i) of the transposed-order backward call for selected chunk i of k (list of float)."""
    sel = (C.c_int32 * max(len(selected), 1))(*[int(x) for x in selected])
    w = (C.c_float * (int(k) - int(i)))() if k > i else (C.c_float * 1)()
    _check(load_library().spaco_gather_row_weights(sel, len(selected), int(i), int(k), float(factor), w),
           "spaco_gather_row_weights")
    return list(w)


# "bwd": dQ and dK/dV in one launch (fp32, short bf16 calls), which then has no "dq" or "dkdv"
PROFILE_KINDS = ("fwd", "bwd", "dq", "dkdv", "kvgrad", "merge")


def _profile_mask(kinds):
    """Bits of the named kinds.  "delta" (rowsum(dO * O), once a kernel) is still taken: nothing is timed for it."""
    return sum(1 << PROFILE_KINDS.index(k) for k in set(kinds) if k != "delta")


def seco_launch_plan(desc, n_col_tiles):
    """(splits per row tile, row tiles, shared-out cache tiles per (batch, KV head), workgroups per such tile) by the general
    planning rules; include/seco.h says which calls follow rules of their own."""
    out = (C.c_int32 * 4)()
    _check(load_library().seco_launch_plan(C.byref(desc), int(n_col_tiles), out), "seco_launch_plan")
    return tuple(out)


def seco_device_info():
    """(compute units, maximum engine clock in kHz) of the current HIP device."""
    cus, khz = C.c_int32(0), C.c_int32(0)
    _check(load_library().seco_device_info(C.byref(cus), C.byref(khz)), "seco_device_info")
    return cus.value, khz.value


def seco_profile_enable(on=True, kinds=None):
    """Time every kernel launch (on=True), none (False), or only the named kinds (subset of PROFILE_KINDS)."""
    if kinds is not None:
        _check(load_library().seco_profile_enable_kinds(_profile_mask(kinds)), "seco_profile_enable_kinds")
    else:
        _check(load_library().seco_profile_enable(1 if on else 0), "seco_profile_enable")


def seco_profile_set(kinds=None):
    """Change which kinds are timed (None: all, []: none) without dropping what has been recorded."""
    mask = _profile_mask(PROFILE_KINDS if kinds is None else kinds)
    _check(load_library().seco_profile_set_kinds(mask), "seco_profile_set_kinds")


def seco_profile_read():
    """{kind: (total_ms, launches)} of the kernels launched since profiling was enabled / last read."""
    ms = (C.c_double * len(PROFILE_KINDS))()
    n = (C.c_int64 * len(PROFILE_KINDS))()
    _check(load_library().seco_profile_read(ms, n), "seco_profile_read")
    return {**{k: (ms[i], n[i]) for i, k in enumerate(PROFILE_KINDS)}, "delta": (0.0, 0)}
