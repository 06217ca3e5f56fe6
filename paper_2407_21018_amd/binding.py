"""ctypes binding of libthk.so: same names as the C ABI, argument marshalling only.

Tensors are torch tensors on the GPU (or raw integer device addresses); PyTorch
supplies device memory and the HIP stream, nothing else.  There is no fallback:
if the library is missing, loading raises.
"""
import ctypes
import os
import struct
import warnings

_HERE = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_HERE, "libthk.so")

THK_F32, THK_BF16 = 0, 1
THK_OP_SCORE, THK_OP_DECODE, THK_OP_PRUNE, THK_OP_SCORE_VALUE, THK_OP_PRUNE_VALUE = 0, 1, 2, 3, 4


class ThkError(RuntimeError):
    def __init__(self, status, where):
        self.status = int(status)
        super().__init__(f"{where}: {thk_status_string(status)} (status {int(status)})")


class thk_shape(ctypes.Structure):
    _fields_ = [("L", ctypes.c_int32), ("B", ctypes.c_int32), ("N_q", ctypes.c_int32),
                ("N_kv", ctypes.c_int32), ("D", ctypes.c_int32), ("S", ctypes.c_int64),
                ("S_obs", ctypes.c_int32), ("T", ctypes.c_int32), ("ld_keep", ctypes.c_int32),
                ("dtype", ctypes.c_int32), ("n_split", ctypes.c_int32), ("S_recent", ctypes.c_int32),
                ("S_cap", ctypes.c_int64)]


_lib = None
_call = None   # the native issue of the per-token calls (csrc/thk_call.cpp), once the library is loaded


def lib_path():
    return _LIB_PATH


def load():
    """Load libthk.so; raises if it has not been built (no CPU fallback exists)."""
    global _lib, _call
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise ImportError(f"{_LIB_PATH} is missing: build it with __graft_entry__.build()")
    # PyTorch's wheel carries its own copy of the HIP runtime.  Loading torch first makes libthk
    # bind to that same copy; loaded the other way round the process ends up with two runtimes
    # and the second one finds no device.
    import torch  # noqa: F401
    L = ctypes.CDLL(_LIB_PATH)
    sp, vp, i32 = ctypes.POINTER(thk_shape), ctypes.c_void_p, ctypes.c_int32
    L.thk_version.restype = i32
    L.thk_version.argtypes = []
    L.thk_reload_env.restype = None
    L.thk_reload_env.argtypes = []
    L.thk_status_string.restype = ctypes.c_char_p
    L.thk_status_string.argtypes = [ctypes.c_int]
    L.thk_last_hip_error.restype = ctypes.c_char_p
    L.thk_last_hip_error.argtypes = []
    L.thk_keep_count.restype = i32
    L.thk_keep_count.argtypes = [i32, ctypes.c_double]
    L.thk_workspace_bytes.restype = ctypes.c_size_t
    L.thk_workspace_bytes.argtypes = [sp, i32]
    L.thk_default_split.restype = i32
    L.thk_default_split.argtypes = [sp, i32]
    L.thk_prune_is_fused.restype = i32
    L.thk_prune_is_fused.argtypes = [sp]
    L.thk_prune_launches.restype = i32
    L.thk_prune_launches.argtypes = [sp]
    L.thk_decode_on_matrix_cores.restype = i32
    L.thk_decode_on_matrix_cores.argtypes = [sp, i32, i32]
    L.thk_score.restype = ctypes.c_int
    L.thk_score.argtypes = [sp, vp, vp, vp, vp, ctypes.c_size_t, vp]
    L.thk_score_value.restype = ctypes.c_int
    L.thk_score_value.argtypes = [sp, vp, vp, vp, i32, vp, vp, ctypes.c_size_t, vp]
    L.thk_prune_value.restype = ctypes.c_int
    L.thk_prune_value.argtypes = [sp, vp, vp, vp, i32, vp, vp, vp, vp, ctypes.c_size_t, vp]
    L.thk_score_magnitude.restype = ctypes.c_int
    L.thk_score_magnitude.argtypes = [sp, vp, i32, vp, vp, ctypes.c_size_t, vp]
    L.thk_select_topk.restype = ctypes.c_int
    L.thk_select_topk.argtypes = [sp, vp, vp, vp]
    L.thk_compact_keys.restype = ctypes.c_int
    L.thk_compact_keys.argtypes = [sp, vp, vp, vp, vp]
    L.thk_prune.restype = ctypes.c_int
    L.thk_prune.argtypes = [sp, vp, vp, vp, vp, vp, vp, ctypes.c_size_t, vp]
    L.thk_decode_attn.restype = ctypes.c_int
    L.thk_decode_attn.argtypes = [sp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp, ctypes.c_size_t, vp]
    L.thk_decode_attn_static.restype = ctypes.c_int
    L.thk_decode_attn_static.argtypes = [sp, vp, vp, vp, vp, vp, vp, i32, i32, vp, vp]
    i64 = ctypes.c_int64
    L.thk_decode_attn_kv.restype = ctypes.c_int
    L.thk_decode_attn_kv.argtypes = [sp, vp, vp, vp, vp, vp, i32, i32, vp, vp, i32, i32, vp, vp,
                                     ctypes.c_size_t, vp]
    L.thk_compact_rows.restype = ctypes.c_int
    L.thk_compact_rows.argtypes = [sp, vp, i64, i64, vp, vp, i64, i64, vp]
    L.thk_copy_rows.restype = ctypes.c_int
    L.thk_copy_rows.argtypes = [sp, vp, i64, i64, vp, i64, i64, i64, vp]
    L.thk_cache_append.restype = ctypes.c_int
    L.thk_cache_append.argtypes = [sp, vp, vp, vp, vp, i32, i32, vp]
    L.thk_tail_flush.restype = ctypes.c_int
    L.thk_tail_flush.argtypes = [sp, vp, vp, vp, vp, vp, i32, i32, i32, vp]
    L.thk_bench_stream.restype = ctypes.c_int
    L.thk_bench_stream.argtypes = [i32, vp, vp, ctypes.c_int64, i32, vp]
    L.thk_profile_next.restype = None
    L.thk_profile_next.argtypes = [vp, vp]
    L.thk_tail_append.restype = ctypes.c_int
    L.thk_tail_append.argtypes = [sp, vp, vp, vp, vp, i32, i32, vp]
    try:   # built for one interpreter and one torch; the library needs neither, and ctypes issues every call
        from . import _thk_call
        addr = lambda f: ctypes.cast(f, vp).value
        _thk_call.bind(addr(L.thk_decode_attn), addr(L.thk_decode_attn_kv), addr(L.thk_tail_append), addr(L.thk_prune), thk_shape)
        _call = _thk_call
    except ImportError as e:
        warnings.warn(f"the native issue of the per-token calls cannot be loaded ({e}): calls go through ctypes, 2 us slower "
                      "each; __graft_entry__.build() builds it", RuntimeWarning, stacklevel=2)
    _lib = L
    return L


def make_shape(L, B, N_q, N_kv, D, S, S_obs, T, ld_keep=0, dtype=THK_BF16, n_split=0, S_recent=0, S_cap=0):
    return thk_shape(L, B, N_q, N_kv, D, S, S_obs, T, ld_keep, dtype, n_split, S_recent, S_cap)


# The calls below are issued once per layer and token, and on short contexts the kernels behind
# them take less than ten microseconds: what a call costs the host decides there.  So a tensor is
# looked at once (one helper checks it and returns its address as a plain int), the shape's
# fields are read in one go, and the current stream's handle comes from torch's raw getter
# (torch.cuda.current_stream() builds a Stream object first).  Decode, append and prune go through
# csrc/thk_call.cpp, which does the same natively for contiguous tensors and leaves everything else (returns
# -1) to the code here.

_FIELDS = struct.Struct("@iiiiiqiiiiiiq")
assert _FIELDS.size == ctypes.sizeof(thk_shape)


def _ptr(x):
    """Device address of a torch tensor (or pass an int / None through)."""
    if x is None or isinstance(x, int):
        return x
    return x.data_ptr()


def _ws(ws):
    """(address, bytes) of a workspace: a tensor, None, or such a pair."""
    if ws is None:
        return None, 0
    if isinstance(ws, tuple):
        return _ptr(ws[0]), ws[1]
    return _ptr(ws), ws.numel() * ws.element_size()


_raw_stream = None   # torch's raw getters, once the runtime is up (see _current_stream)


def _forget_runtime():
    global _raw_stream
    _raw_stream = None
    if _call is not None:
        _call.stream_getters(None, None)


os.register_at_fork(after_in_child=_forget_runtime)   # a forked child must go through torch's own checks


def _current_stream():
    global _raw_stream
    if _raw_stream is not None:
        get_stream, get_device = _raw_stream
        return get_stream(get_device())
    import torch
    handle = torch.cuda.current_stream().cuda_stream   # initialises the runtime, or raises
    get_stream = getattr(torch._C, "_cuda_getCurrentRawStream", None)
    get_device = getattr(torch._C, "_cuda_getDevice", None)
    if get_stream is not None and get_device is not None:
        _raw_stream = (get_stream, get_device)
        load()
        if _call is not None:
            _call.stream_getters(get_stream, get_device)
    return handle


def _stream(stream):
    if stream is None:
        return _current_stream()
    if isinstance(stream, int):
        return stream
    return stream.cuda_stream


def _arg(x, n, name, where):
    """Address of a tensor, after a host-side guard: a tensor handed to a kernel must hold at
    least the n elements the shape implies (a short tensor would make the kernel read or write
    out of bounds)."""
    if x is None or isinstance(x, int):
        return x
    if x.numel() < n:
        raise ValueError(f"{where}: {name} holds {x.numel()} elements, the shape needs {n}")
    if not x.is_contiguous():
        raise ValueError(f"{where}: {name} must be contiguous")
    return x.data_ptr()


def _dims(s):
    """(units, query heads, D, S, S_obs, T, row pitch, S_recent, S_cap) of a shape."""
    L, B, N_q, N_kv, D, S, S_obs, T, ld, _, _, S_recent, S_cap = _FIELDS.unpack_from(s)
    LB = L * B
    return LB * N_kv, LB * N_q, D, S, S_obs, T, ld or T, S_recent, S_cap


def thk_last_hip_error():
    return load().thk_last_hip_error().decode()


def _issued(st, where):
    """True when the native code took the call, whose status is then checked."""
    if st == 0:
        return True
    if st < 0:
        return False
    _check(st, where)


def _check(st, where):
    if st == 6:
        raise ThkError(st, f"{where} [{thk_last_hip_error()}]")
    if st != 0:
        raise ThkError(st, where)


def thk_version():
    return int(load().thk_version())


def thk_reload_env():
    """Make the library read its THK_* environment switches again (it reads them once per process)."""
    load().thk_reload_env()


def thk_status_string(st):
    return load().thk_status_string(int(st)).decode()


def thk_keep_count(D, lam):
    return int(load().thk_keep_count(D, lam))


def thk_workspace_bytes(shape, op):
    return int(load().thk_workspace_bytes(ctypes.byref(shape), op))


def thk_default_split(shape, op):
    return int(load().thk_default_split(ctypes.byref(shape), op))


def thk_prune_is_fused(shape):
    return int(load().thk_prune_is_fused(ctypes.byref(shape)))


def thk_prune_launches(shape):
    return int(load().thk_prune_launches(ctypes.byref(shape)))


def thk_decode_on_matrix_cores(shape, T_v=0, ld_v=0):
    return int(load().thk_decode_on_matrix_cores(ctypes.byref(shape), T_v, ld_v))


def thk_score(shape, q_obs, k, score, ws, stream=None):
    w = "thk_score"
    U, H, D, S, S_obs, _, _, _, _ = _dims(shape)
    _check(load().thk_score(ctypes.byref(shape), _arg(q_obs, H * S_obs * D, "q_obs", w), _arg(k, U * S * D, "k", w),
                            _arg(score, U * D, "score", w), *_ws(ws), _stream(stream)), w)


def thk_score_value(shape, q_obs, k, v, causal, score_v, ws, stream=None):
    w = "thk_score_value"
    U, H, D, S, S_obs, _, _, _, _ = _dims(shape)
    _check(load().thk_score_value(ctypes.byref(shape), _arg(q_obs, H * S_obs * D, "q_obs", w),
                                  _arg(k, U * S * D, "k", w), _arg(v, U * S * D, "v", w), int(causal),
                                  _arg(score_v, U * D, "score_v", w), *_ws(ws), _stream(stream)), w)


def thk_prune_value(shape, q_obs, k, v, causal, score_v, idx_v, v_pruned, ws, stream=None):
    w = "thk_prune_value"
    U, H, D, S, S_obs, T, ld, S_recent, S_cap = _dims(shape)
    _check(load().thk_prune_value(ctypes.byref(shape), _arg(q_obs, H * S_obs * D, "q_obs", w),
                                  _arg(k, U * S * D, "k", w), _arg(v, U * S * D, "v", w), int(causal),
                                  _arg(score_v, U * D, "score_v", w), _arg(idx_v, U * T, "idx_v", w),
                                  _arg(v_pruned, U * (S_cap or S - S_recent) * ld, "v_pruned", w), *_ws(ws),
                                  _stream(stream)), w)


def thk_score_magnitude(shape, k, p, score, ws, stream=None):
    w = "thk_score_magnitude"
    U, _, D, S, _, _, _, _, _ = _dims(shape)
    _check(load().thk_score_magnitude(ctypes.byref(shape), _arg(k, U * S * D, "k", w), p,
                                      _arg(score, U * D, "score", w), *_ws(ws), _stream(stream)), w)


def thk_select_topk(shape, score, idx, stream=None):
    w = "thk_select_topk"
    U, _, D, _, _, T, _, _, _ = _dims(shape)
    _check(load().thk_select_topk(ctypes.byref(shape), _arg(score, U * D, "score", w), _arg(idx, U * T, "idx", w),
                                  _stream(stream)), w)


def thk_compact_keys(shape, k, idx, k_pruned, stream=None):
    w = "thk_compact_keys"
    U, _, D, S, _, T, ld, S_recent, S_cap = _dims(shape)
    _check(load().thk_compact_keys(ctypes.byref(shape), _arg(k, U * S * D, "k", w), _arg(idx, U * T, "idx", w),
                                   _arg(k_pruned, U * (S_cap or S - S_recent) * ld, "k_pruned", w), _stream(stream)), w)


def thk_prune(shape, q_obs, k, score, idx, k_pruned, ws, stream=None):
    w = "thk_prune"
    if _call is not None and _issued(_call.prune(shape, q_obs, k, score, idx, k_pruned, ws, stream), w):
        return
    U, H, D, S, S_obs, T, ld, S_recent, S_cap = _dims(shape)
    _check(load().thk_prune(ctypes.byref(shape), _arg(q_obs, H * S_obs * D, "q_obs", w), _arg(k, U * S * D, "k", w),
                            _arg(score, U * D, "score", w), _arg(idx, U * T, "idx", w),
                            _arg(k_pruned, U * (S_cap or S - S_recent) * ld, "k_pruned", w), *_ws(ws),
                            _stream(stream)), w)


def _tail_args(k_tail, v_tail, n, s_tail, w):
    """Addresses of the tail tensors; without tail rows they are not looked at."""
    if s_tail > 0:
        return _arg(k_tail, n, "k_tail", w), _arg(v_tail, n, "v_tail", w)
    return _ptr(k_tail), _ptr(v_tail)


def thk_decode_attn(shape, q, k_pruned, idx, v, k_tail, v_tail, s_tail, s_tail_cap, out, ws,
                    stream=None):
    w = "thk_decode_attn"
    if _call is not None and _issued(_call.decode_attn(shape, q, k_pruned, idx, v, k_tail, v_tail, s_tail, s_tail_cap, out, ws,
                                                       stream), w):
        return
    U, H, D, S, _, T, ld, _, S_cap = _dims(shape)
    n, rows = H * D, U * (S_cap or S)
    qp, op = _arg(q, n, "q", w), _arg(out, n, "out", w)
    kp, ip, vp = _arg(k_pruned, rows * ld, "k_pruned", w), _arg(idx, U * T, "idx", w), _arg(v, rows * D, "v", w)
    kt, vt = _tail_args(k_tail, v_tail, U * s_tail_cap * D, s_tail, w)
    _check(load().thk_decode_attn(ctypes.byref(shape), qp, kp, ip, vp, kt, vt, s_tail, s_tail_cap, op, *_ws(ws),
                                  _stream(stream)), w)


def thk_decode_attn_static(shape, q, k_pruned, idx, v, k_tail, v_tail, s_tail, s_tail_cap, out, stream=None):
    w = "thk_decode_attn_static"
    U, H, D, S, _, T, ld, _, S_cap = _dims(shape)
    n, rows = H * D, U * (S_cap or S)
    qp, op = _arg(q, n, "q", w), _arg(out, n, "out", w)
    kp, ip, vp = _arg(k_pruned, rows * ld, "k_pruned", w), _arg(idx, U * T, "idx", w), _arg(v, rows * D, "v", w)
    kt, vt = _tail_args(k_tail, v_tail, U * s_tail_cap * D, s_tail, w)
    _check(load().thk_decode_attn_static(ctypes.byref(shape), qp, kp, ip, vp, kt, vt, s_tail, s_tail_cap, op,
                                         _stream(stream)), w)


def thk_decode_attn_kv(shape, q, k_pruned, idx, v_pruned, idx_v, T_v, ld_v, k_tail, v_tail, s_tail,
                       s_tail_cap, out, ws, stream=None):
    w = "thk_decode_attn_kv"
    if _call is not None and _issued(_call.decode_attn_kv(shape, q, k_pruned, idx, v_pruned, idx_v, T_v, ld_v, k_tail, v_tail,
                                                          s_tail, s_tail_cap, out, ws, stream), w):
        return
    U, H, D, S, _, T, ld, _, S_cap = _dims(shape)
    n, rows = H * D, U * (S_cap or S)
    qp, op = _arg(q, n, "q", w), _arg(out, n, "out", w)
    kp, ip = _arg(k_pruned, rows * ld, "k_pruned", w), _arg(idx, U * T, "idx", w)
    vp, ivp = _arg(v_pruned, rows * max(ld_v, 0), "v_pruned", w), _arg(idx_v, U * max(T_v, 0), "idx_v", w)
    kt, vt = _tail_args(k_tail, v_tail, U * s_tail_cap * D, s_tail, w)
    _check(load().thk_decode_attn_kv(ctypes.byref(shape), qp, kp, ip, vp, ivp, T_v, ld_v, kt, vt, s_tail, s_tail_cap,
                                     op, *_ws(ws), _stream(stream)), w)


def thk_tail_append(shape, k_new, v_new, k_tail, v_tail, s_tail, s_tail_cap, stream=None):
    w = "thk_tail_append"
    if _call is not None and _issued(_call.tail_append(shape, k_new, v_new, k_tail, v_tail, s_tail, s_tail_cap, stream), w):
        return
    U, _, D, _, _, _, _, _, _ = _dims(shape)
    n, m = U * D, U * s_tail_cap * D
    _check(load().thk_tail_append(ctypes.byref(shape), _arg(k_new, n, "k_new", w), _arg(v_new, n, "v_new", w),
                                  _arg(k_tail, m, "k_tail", w), _arg(v_tail, m, "v_tail", w), s_tail, s_tail_cap,
                                  _stream(stream)), w)


def thk_compact_rows(shape, src, src_unit_rows, src_row0, idx, k_pruned, dst_row0, n_rows, stream=None):
    w = "thk_compact_rows"
    U, _, D, S, _, T, ld, _, S_cap = _dims(shape)
    _check(load().thk_compact_rows(ctypes.byref(shape), _arg(src, U * src_unit_rows * D, "src", w), src_unit_rows,
                                   src_row0, _arg(idx, U * T, "idx", w),
                                   _arg(k_pruned, U * (S_cap or S) * ld, "k_pruned", w), dst_row0, n_rows,
                                   _stream(stream)), w)


def thk_copy_rows(shape, src, src_unit_rows, src_row0, dst, dst_unit_rows, dst_row0, n_rows, stream=None):
    w = "thk_copy_rows"
    U, _, D, _, _, _, _, _, _ = _dims(shape)
    _check(load().thk_copy_rows(ctypes.byref(shape), _arg(src, U * src_unit_rows * D, "src", w), src_unit_rows,
                                src_row0, _arg(dst, U * dst_unit_rows * D, "dst", w), dst_unit_rows, dst_row0, n_rows,
                                _stream(stream)), w)


def thk_cache_append(shape, k_new, v_new, k_tail, v, s_tail, s_tail_cap, stream=None):
    w = "thk_cache_append"
    U, _, D, S, _, _, _, _, S_cap = _dims(shape)
    n = U * D
    _check(load().thk_cache_append(ctypes.byref(shape), _arg(k_new, n, "k_new", w), _arg(v_new, n, "v_new", w),
                                   _arg(k_tail, U * s_tail_cap * D, "k_tail", w), _arg(v, U * (S_cap or S) * D, "v", w),
                                   s_tail, s_tail_cap, _stream(stream)), w)


def thk_tail_flush(shape, idx, k_pruned, k_tail, v, v_tail, s_tail, s_tail_cap, n_flush, stream=None):
    w = "thk_tail_flush"
    U, _, D, S, _, T, ld, _, S_cap = _dims(shape)
    rows, m = U * (S_cap or S), U * s_tail_cap * D
    _check(load().thk_tail_flush(ctypes.byref(shape), _arg(idx, U * T, "idx", w), _arg(k_pruned, rows * ld, "k_pruned", w),
                                 _arg(k_tail, m, "k_tail", w), _arg(v, rows * D, "v", w), _arg(v_tail, m, "v_tail", w),
                                 s_tail, s_tail_cap, n_flush, _stream(stream)), w)


THK_STREAM_READ, THK_STREAM_COPY, THK_STREAM_WRITE = 0, 1, 2


def thk_bench_stream(mode, src, dst, n_blocks, w, stream=None):
    """Plain read / copy / write stream for benchmarks: n_blocks blocks of 128 KiB of src and
    w * 4 KiB of dst each (src or dst may be None where the mode does not use it)."""
    if src is not None:
        _arg(src, n_blocks * 131072 // src.element_size(), "src", "thk_bench_stream")
    if dst is not None and mode != THK_STREAM_READ:
        _arg(dst, n_blocks * w * 4096 // dst.element_size(), "dst", "thk_bench_stream")
    _check(load().thk_bench_stream(mode, _ptr(src), _ptr(dst), n_blocks, w, _stream(stream)), "thk_bench_stream")


def thk_profile_next(ev_start, ev_stop):
    """ev_start / ev_stop: torch.cuda.Event(enable_timing=True) that have been recorded once
    (torch creates the HIP event lazily), raw hipEvent_t integers, or None to cancel."""
    def h(e):
        if e is None or isinstance(e, int):
            return e
        return e.cuda_event
    load().thk_profile_next(ctypes.c_void_p(h(ev_start)) if ev_start is not None else None,
                            ctypes.c_void_p(h(ev_stop)) if ev_stop is not None else None)
