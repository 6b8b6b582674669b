"""Thin ctypes binding of liblaserkv.so: argument marshalling only.

Every step of the path runs in the library's HIP kernels.  There is no CPU
fallback: loading fails loudly when the library has not been built.
PyTorch is used by callers for device memory and streams; this module only
reads `data_ptr()`, strides and the current stream handle.
"""
from __future__ import annotations

import ctypes as C
import os

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "liblaserkv.so")

LKV_F32, LKV_BF16 = 0, 1
LKV_OK, LKV_EINVAL, LKV_ECAP, LKV_ENOMEM, LKV_EHIP = 0, -1, -2, -3, -4
LKV_WINDOW_AT_BLOCK_END = -(1 << 63)   # q_pos0 sentinel of laserkv.h

EXPORTS = (
    "laserkv_create", "laserkv_destroy", "laserkv_last_error", "laserkv_budget",
    "laserkv_partition", "laserkv_select_block", "laserkv_append", "laserkv_compress_block",
    "laserkv_profile_begin", "laserkv_profile_end", "laserkv_profile_isolate", "laserkv_layer_plan",
    "laserkv_score_block", "laserkv_select_consensus", "laserkv_append_shared", "laserkv_set_row_lse",
    "laserkv_set_row_lse_complete", "laserkv_attend_workspace_bytes", "laserkv_attend_cache",
    "laserkv_attend_block_workspace_bytes", "laserkv_attend_block",
    "laserkv_layer_workspace_bytes", "laserkv_compress_layer",
    "laserkv_static_init", "laserkv_static_workspace_bytes", "laserkv_compress_block_static",
)
LKV_STATIC_SCRATCH_BYTES = 32 << 20
LAYER_PLAN = ("stat_ranges", "stat_keys", "score_ranges", "score_keys", "copied_rows")
KERNEL_NAMES = ("sweep1", "sweep2", "count", "select", "append", "attend", "single")


class LaserKVError(RuntimeError):
    def __init__(self, code: int, msg: str):
        super().__init__(f"laserkv error {code}: {msg}")
        self.code = code


class Config(C.Structure):
    _fields_ = [(n, C.c_int32) for n in (
        "n_q_heads", "n_kv_heads", "head_dim", "dtype", "lsh_tables", "lsh_bits",
        "max_block", "max_window", "max_ctx_keys")]


_lib = None


def load():
    """Load the built library (never builds, never falls back)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise RuntimeError(
            f"{LIB_PATH} is missing: build it first with `python -m paper_2602_02199_amd.build` "
            "(there is no CPU fallback)")
    lib = C.CDLL(LIB_PATH)
    vp, i32, i64 = C.c_void_p, C.c_int32, C.c_int64
    lib.laserkv_create.argtypes = [C.POINTER(Config), C.POINTER(vp)]
    lib.laserkv_create.restype = C.c_int
    lib.laserkv_destroy.argtypes = [vp]
    lib.laserkv_destroy.restype = None
    lib.laserkv_last_error.argtypes = [vp]
    lib.laserkv_last_error.restype = C.c_char_p
    lib.laserkv_budget.argtypes = [i64, i64, i64, i64]
    lib.laserkv_budget.restype = i64
    lib.laserkv_partition.argtypes = [i32, i32, C.c_double, i32] + [C.POINTER(i32)] * 4
    lib.laserkv_partition.restype = C.c_int
    lib.laserkv_select_block.argtypes = [
        vp, vp, i64, i64, vp, i64, i64, vp, i64, i64, vp,
        i32, i32, i32, i64, i64, i32, i32, i32, i32, i32,
        vp, vp, vp, vp, vp, vp]
    lib.laserkv_select_block.restype = C.c_int
    lib.laserkv_append.argtypes = [
        vp, vp, i64, i64, vp, i64, i64, vp, i32, i32, i64,
        vp, vp, i64, vp, i64, i64, i64, vp]
    lib.laserkv_append.restype = C.c_int
    lib.laserkv_compress_block.argtypes = [
        vp, vp, i64, i64, vp, i64, i64, vp, i64, i64, vp, i64, i64, vp,
        i32, i32, i32, i64, i64, i32, i32, i32, i32, i32,
        vp, vp, vp, i64, vp, i64, i64, i64, vp]
    lib.laserkv_compress_block.restype = C.c_int
    lib.laserkv_layer_workspace_bytes.argtypes = [vp, i64, i32, i32, i32]
    lib.laserkv_layer_workspace_bytes.restype = i64
    lib.laserkv_compress_layer.argtypes = [vp, vp, i64, i64, i64, vp, i64, i64, vp, i64, i64, vp, i64, i32, i32,
                                           i32, i32, C.c_double, vp, vp, vp, vp, i64, vp, i64, i64, vp, i64, vp]
    lib.laserkv_compress_layer.restype = C.c_int
    lib.laserkv_static_init.argtypes = []
    lib.laserkv_static_init.restype = C.c_int
    lib.laserkv_static_workspace_bytes.argtypes = [C.POINTER(Config)]
    lib.laserkv_static_workspace_bytes.restype = C.c_size_t
    lib.laserkv_compress_block_static.argtypes = [C.POINTER(Config)] + lib.laserkv_compress_block.argtypes[1:]
    lib.laserkv_compress_block_static.restype = C.c_int
    lib.laserkv_score_block.argtypes = [
        vp, vp, i64, i64, vp, i64, i64, vp, i64, i64, vp,
        i32, i32, i32, i64, i64, i32, vp, vp, i32, vp]
    lib.laserkv_score_block.restype = C.c_int
    lib.laserkv_select_consensus.argtypes = [vp, vp, vp, i32, i32, i32, i32, i32, vp, vp]
    lib.laserkv_select_consensus.restype = C.c_int
    lib.laserkv_append_shared.argtypes = lib.laserkv_append.argtypes
    lib.laserkv_append_shared.restype = C.c_int
    lib.laserkv_set_row_lse.argtypes = [vp, vp]
    lib.laserkv_set_row_lse.restype = C.c_int
    lib.laserkv_set_row_lse_complete.argtypes = [vp, vp]
    lib.laserkv_set_row_lse_complete.restype = C.c_int
    lib.laserkv_attend_workspace_bytes.argtypes = [vp, i32, i64]
    lib.laserkv_attend_workspace_bytes.restype = i64
    lib.laserkv_attend_cache.argtypes = [vp, vp, i64, i64, i32, vp, vp, i64, i64, vp, vp, vp, i64, vp]
    lib.laserkv_attend_cache.restype = C.c_int
    lib.laserkv_attend_block_workspace_bytes.argtypes = [vp, i32, i64, i32]
    lib.laserkv_attend_block_workspace_bytes.restype = i64
    lib.laserkv_attend_block.argtypes = [vp, vp, i64, i64, i32, vp, vp, i64, i64, vp, i64, i64, vp, i64, i64,
                                         i32, i64, i64, i32, vp, vp, vp, i64, vp]
    lib.laserkv_attend_block.restype = C.c_int
    lib.laserkv_profile_begin.argtypes = [vp]
    lib.laserkv_profile_begin.restype = C.c_int
    lib.laserkv_profile_end.argtypes = [vp, C.POINTER(C.c_double), C.POINTER(i64)]
    lib.laserkv_profile_end.restype = C.c_int
    lib.laserkv_profile_isolate.argtypes = [vp, i32]
    lib.laserkv_profile_isolate.restype = C.c_int
    lib.laserkv_layer_plan.argtypes = [vp, i64, i32, i32, i32, i32, C.c_double, i32, C.POINTER(i64)]
    lib.laserkv_layer_plan.restype = C.c_int
    _lib = lib
    return lib


def laserkv_budget(s_block: int, l_ctx: int, r_num: int = 1, r_den: int = 4) -> int:
    b = load().laserkv_budget(s_block, l_ctx, r_num, r_den)
    if b < 0:
        raise LaserKVError(LKV_EINVAL, "budget: bad arguments")
    return int(b)


def laserkv_partition(B: int, n: int, alpha: float, s_t: int):
    lib = load()
    out = [C.c_int32() for _ in range(4)]
    rc = lib.laserkv_partition(B, n, alpha, s_t, *[C.byref(o) for o in out])
    if rc != LKV_OK:
        raise LaserKVError(rc, lib.laserkv_last_error(None).decode())
    return tuple(int(o.value) for o in out)


def laserkv_static_init():
    lib = load()
    rc = lib.laserkv_static_init()
    if rc != LKV_OK:
        raise LaserKVError(rc, lib.laserkv_last_error(None).decode())


def laserkv_static_workspace_bytes(cfg: Config) -> int:
    return int(load().laserkv_static_workspace_bytes(C.byref(cfg)))


def laserkv_compress_block_static(cfg: Config, q_win, k_blk, v_blk, k_ctx, hyperplanes, *, block_pos0, q_pos0=None,
                                  causal=True, n_anchor, n_local, k_exact, k_lsh, keep_idx, k_cache, v_cache, cache_pos,
                                  cache_len, stream):
    """laserkv_compress_block on the library's static scratch (no context, no allocation).  stream: raw handle."""
    lib = load()
    d = cfg.head_dim
    q, qsh, qst, w = _rows3(q_win, d)
    k, ksh, kst, s_t = _rows3(k_blk, d)
    v, vsh, vst, _ = _rows3(v_blk, d)
    c, csh, cst, t_ctx = _context3(k_ctx, d)
    kc, vc, cache_sh, cap = _cache(k_cache, v_cache, d)
    assert hyperplanes.is_contiguous()
    rc = lib.laserkv_compress_block_static(
        C.byref(cfg), q, qsh, qst, k, ksh, kst, v, vsh, vst, c, csh, cst, hyperplanes.data_ptr(), s_t, w, t_ctx, block_pos0,
        LKV_WINDOW_AT_BLOCK_END if q_pos0 is None else q_pos0, 1 if causal else 0, n_anchor, n_local, k_exact, k_lsh,
        _ptr(keep_idx), kc, vc, cache_sh, _ptr(cache_pos), cache_pos.stride(0), cache_len, cap, stream)
    if rc != LKV_OK:
        raise LaserKVError(rc, lib.laserkv_last_error(None).decode())


# Small calls cost what their marshalling costs: every attribute of a tensor is read once (about 0.1 us each), addresses
# go to ctypes as plain integers.
def _ptr(t):
    return None if t is None else t.data_ptr()


def _rows3(t, d):
    """(address, head stride, row stride, rows) of a [heads, rows, d] tensor with d contiguous."""
    sh, st, one = t.stride()
    _, n, dd = t.shape
    assert one == 1 and dd == d, "expected [heads, rows, d] with d contiguous"
    return t.data_ptr(), sh, st, n


def _rows4(t, d):
    """(address, block stride, head stride, row stride, blocks, rows) of a [blocks, heads, rows, d] tensor with d contiguous."""
    sb, sh, st, one = t.stride()
    nb, _, n, dd = t.shape
    assert one == 1 and dd == d, "expected [blocks, heads, rows, d] with d contiguous"
    return t.data_ptr(), sb, sh, st, nb, n


def _context3(t, d):
    return (None, 0, 0, 0) if t is None else _rows3(t, d)


def _cache(k_cache, v_cache, d):
    """(K address, V address, head stride, capacity) of a cache pair [H_kv, cap, d] with contiguous rows."""
    ks = k_cache.stride()
    assert ks[2] == 1 and ks[1] == d and v_cache.stride() == ks
    return k_cache.data_ptr(), v_cache.data_ptr(), ks[0], k_cache.shape[1]


class LaserKV:
    """One library context (owns the device workspace).  Methods mirror the C entry points."""

    def __init__(self, n_q_heads, n_kv_heads, head_dim, dtype, lsh_tables, lsh_bits,
                 max_block, max_window, max_ctx_keys):
        import torch
        self._lib = load()
        self._torch = torch
        if not torch.cuda.is_available():
            raise RuntimeError("laserkv needs a GPU: there is no CPU path")
        self.cfg = Config(n_q_heads, n_kv_heads, head_dim,
                          {"f32": LKV_F32, "bf16": LKV_BF16}[dtype] if isinstance(dtype, str) else dtype,
                          lsh_tables, lsh_bits, max_block, max_window, max_ctx_keys)
        self._head_dim = head_dim
        self._raw_stream, self._current_device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice
        self._ctx = C.c_void_p()
        rc = self._lib.laserkv_create(C.byref(self.cfg), C.byref(self._ctx))
        if rc != LKV_OK:
            raise LaserKVError(rc, self._lib.laserkv_last_error(None).decode())

    def close(self):
        if getattr(self, "_ctx", None) is not None and self._ctx:
            self._lib.laserkv_destroy(self._ctx)
            self._ctx = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, rc):
        if rc != LKV_OK:
            raise LaserKVError(rc, self._lib.laserkv_last_error(self._ctx).decode())

    def _stream(self, stream):
        # the raw handle without a Stream object around it (0.3 instead of 2.8 us)
        return self._raw_stream(self._current_device()) if stream is None else stream

    def laserkv_select_block(self, q_win, k_blk, k_ctx, hyperplanes, *, block_pos0, q_pos0=None, causal=True,
                             n_anchor, n_local, k_exact, k_lsh, keep_idx,
                             dbg_s_exact=None, dbg_sig_k=None, dbg_sig_q=None, dbg_count=None, stream=None):
        d = self._head_dim
        q, qsh, qst, w = _rows3(q_win, d)
        k, ksh, kst, s_t = _rows3(k_blk, d)
        c, csh, cst, t_ctx = _context3(k_ctx, d)
        assert hyperplanes.is_contiguous()
        rc = self._lib.laserkv_select_block(
            self._ctx, q, qsh, qst, k, ksh, kst, c, csh, cst, hyperplanes.data_ptr(), s_t, w, t_ctx, block_pos0,
            LKV_WINDOW_AT_BLOCK_END if q_pos0 is None else q_pos0, 1 if causal else 0, n_anchor, n_local, k_exact, k_lsh,
            _ptr(keep_idx), _ptr(dbg_s_exact), _ptr(dbg_sig_k), _ptr(dbg_sig_q), _ptr(dbg_count), self._stream(stream))
        if rc:
            self._check(rc)

    def _append(self, fn, k_blk, v_blk, keep_idx, b_t, block_pos0, k_cache, v_cache, cache_pos, cache_len, stream):
        d = self._head_dim
        k, ksh, kst, s_t = _rows3(k_blk, d)
        v, vsh, vst, _ = _rows3(v_blk, d)
        kc, vc, cache_sh, cap = _cache(k_cache, v_cache, d)
        rc = fn(self._ctx, k, ksh, kst, v, vsh, vst, _ptr(keep_idx), b_t, s_t, block_pos0, kc, vc, cache_sh,
                _ptr(cache_pos), cache_pos.stride(0), cache_len, cap, self._stream(stream))
        if rc:
            self._check(rc)

    def laserkv_append(self, k_blk, v_blk, keep_idx, *, b_t, block_pos0, k_cache, v_cache, cache_pos,
                       cache_len, stream=None):
        self._append(self._lib.laserkv_append, k_blk, v_blk, keep_idx, b_t, block_pos0, k_cache, v_cache, cache_pos,
                     cache_len, stream)

    def laserkv_compress_block(self, q_win, k_blk, v_blk, k_ctx, hyperplanes, *, block_pos0, q_pos0=None, causal=True,
                               n_anchor, n_local, k_exact, k_lsh, keep_idx, k_cache, v_cache, cache_pos, cache_len,
                               stream=None):
        d = self._head_dim
        q, qsh, qst, w = _rows3(q_win, d)
        k, ksh, kst, s_t = _rows3(k_blk, d)
        v, vsh, vst, _ = _rows3(v_blk, d)
        c, csh, cst, t_ctx = _context3(k_ctx, d)
        kc, vc, cache_sh, cap = _cache(k_cache, v_cache, d)
        assert hyperplanes.is_contiguous()
        rc = self._lib.laserkv_compress_block(
            self._ctx, q, qsh, qst, k, ksh, kst, v, vsh, vst, c, csh, cst, hyperplanes.data_ptr(), s_t, w, t_ctx, block_pos0,
            LKV_WINDOW_AT_BLOCK_END if q_pos0 is None else q_pos0, 1 if causal else 0, n_anchor, n_local, k_exact, k_lsh,
            _ptr(keep_idx), kc, vc, cache_sh, _ptr(cache_pos), cache_pos.stride(0), cache_len, cap, self._stream(stream))
        if rc:
            self._check(rc)

    def laserkv_score_block(self, q_win, k_blk, k_ctx, hyperplanes, *, block_pos0, q_pos0=None, causal=True,
                            score_acc, count_acc, accumulate, stream=None):
        d = self._head_dim
        q, qsh, qst, w = _rows3(q_win, d)
        k, ksh, kst, s_t = _rows3(k_blk, d)
        c, csh, cst, t_ctx = _context3(k_ctx, d)
        assert hyperplanes.is_contiguous() and score_acc.is_contiguous() and count_acc.is_contiguous()
        assert score_acc.numel() >= s_t and count_acc.numel() >= s_t
        rc = self._lib.laserkv_score_block(
            self._ctx, q, qsh, qst, k, ksh, kst, c, csh, cst, hyperplanes.data_ptr(), s_t, w, t_ctx, block_pos0,
            LKV_WINDOW_AT_BLOCK_END if q_pos0 is None else q_pos0, 1 if causal else 0,
            score_acc.data_ptr(), count_acc.data_ptr(), 1 if accumulate else 0, self._stream(stream))
        if rc:
            self._check(rc)

    def laserkv_select_consensus(self, score_acc, count_acc, *, s_t, n_anchor, n_local, k_exact, k_lsh, keep_idx,
                                 stream=None):
        assert score_acc.is_contiguous() and count_acc.is_contiguous() and keep_idx.is_contiguous()
        rc = self._lib.laserkv_select_consensus(self._ctx, _ptr(score_acc), _ptr(count_acc), s_t, n_anchor, n_local,
                                                k_exact, k_lsh, _ptr(keep_idx), self._stream(stream))
        self._check(rc)

    def laserkv_append_shared(self, k_blk, v_blk, keep_idx, *, b_t, block_pos0, k_cache, v_cache, cache_pos,
                              cache_len, stream=None):
        self._append(self._lib.laserkv_append_shared, k_blk, v_blk, keep_idx, b_t, block_pos0, k_cache, v_cache, cache_pos,
                     cache_len, stream)

    def laserkv_set_row_lse(self, row_lse):
        """row_lse: contiguous float32 [H_q, w] device tensor, or None to switch the feature off.  The tensor
        is kept alive by this object for as long as it is set."""
        if row_lse is not None:
            assert row_lse.is_contiguous() and row_lse.dtype == self._torch.float32
        self._row_lse = row_lse
        self._check(self._lib.laserkv_set_row_lse(self._ctx, _ptr(row_lse)))

    def laserkv_set_row_lse_complete(self, row_lse):
        """row_lse: contiguous float32 [H_q, w] device tensor holding every window row's complete log-sum-exp,
        or None to let the library compute the statistics itself again."""
        if row_lse is not None:
            assert row_lse.is_contiguous() and row_lse.dtype == self._torch.float32
        self._row_lse = row_lse
        self._check(self._lib.laserkv_set_row_lse_complete(self._ctx, _ptr(row_lse)))

    def laserkv_attend_workspace_bytes(self, n_q, cache_len):
        n = int(self._lib.laserkv_attend_workspace_bytes(self._ctx, n_q, cache_len))
        if n < 0:
            raise LaserKVError(LKV_EINVAL, "attend_workspace_bytes: n_q or cache_len out of range")
        return n

    def laserkv_attend_cache(self, q, k_cache, v_cache, *, cache_len, out, out_lse, workspace, stream=None):
        """q [H_q, n_q, d]; k_cache / v_cache [H_kv, cap, d]; out float32 [H_q, n_q, d] or None (normaliser only),
        out_lse float32 [H_q, n_q];
        workspace: uint8 device tensor of at least laserkv_attend_workspace_bytes(n_q, cache_len) bytes."""
        d = self._head_dim
        qp, qsh, qst, n_q = _rows3(q, d)
        ks = k_cache.stride()
        assert ks[2] == 1 and ks[1] == d and v_cache.stride() == ks
        f32 = self._torch.float32
        shape = q.shape
        assert out is None or (out.is_contiguous() and out.dtype is f32 and out.shape == shape)
        assert out_lse.is_contiguous() and out_lse.dtype is f32 and out_lse.shape == shape[:2]
        assert workspace.is_contiguous() and workspace.element_size() == 1
        rc = self._lib.laserkv_attend_cache(
            self._ctx, qp, qsh, qst, n_q, k_cache.data_ptr(), v_cache.data_ptr(), ks[0], cache_len,
            _ptr(out), out_lse.data_ptr(), workspace.data_ptr(), workspace.numel(), self._stream(stream))
        if rc:
            self._check(rc)

    def laserkv_attend_block_workspace_bytes(self, n_q, cache_len, s_t):
        n = int(self._lib.laserkv_attend_block_workspace_bytes(self._ctx, n_q, cache_len, s_t))
        if n < 0:
            raise LaserKVError(LKV_EINVAL, "attend_block_workspace_bytes: n_q, cache_len or s_t out of range")
        return n

    def laserkv_attend_block(self, q, k_cache, v_cache, k_blk, v_blk, *, cache_len, block_pos0, q_pos0=None, causal=True,
                             out, out_lse, workspace, stream=None):
        """q [H_q, n_q, d]; k_cache / v_cache [H_kv, cap, d] (may be None with cache_len 0); k_blk / v_blk
        [H_kv, s_t, d] (views with strides allowed); out float32 [H_q, n_q, d], out_lse float32 [H_q, n_q];
        q_pos0 defaults to the block's last n_q positions;
        workspace: uint8 device tensor of at least laserkv_attend_block_workspace_bytes(n_q, cache_len, s_t) bytes."""
        d = self._head_dim
        qp, qsh, qst, n_q = _rows3(q, d)
        k, ksh, kst, s_t = _rows3(k_blk, d)
        v, vsh, vst, _ = _rows3(v_blk, d)
        assert v_blk.shape == k_blk.shape
        kc = vc = None
        cache_sh = 0
        if k_cache is not None:
            kc, vc, cache_sh, _ = _cache(k_cache, v_cache, d)
        f32 = self._torch.float32
        shape = q.shape
        assert out.is_contiguous() and out.dtype is f32 and out.shape == shape
        assert out_lse.is_contiguous() and out_lse.dtype is f32 and out_lse.shape == shape[:2]
        assert workspace.is_contiguous() and workspace.element_size() == 1
        rc = self._lib.laserkv_attend_block(
            self._ctx, qp, qsh, qst, n_q, kc, vc, cache_sh, cache_len, k, ksh, kst, v, vsh, vst, s_t, block_pos0,
            block_pos0 + s_t - n_q if q_pos0 is None else q_pos0, 1 if causal else 0,
            out.data_ptr(), out_lse.data_ptr(), workspace.data_ptr(), workspace.numel(), self._stream(stream))
        if rc:
            self._check(rc)

    def laserkv_profile_begin(self):
        self._check(self._lib.laserkv_profile_begin(self._ctx))

    def laserkv_profile_end(self):
        """Returns {kernel name: (total ms, launches)}."""
        n = len(KERNEL_NAMES)
        ms = (C.c_double * n)()
        cnt = (C.c_int64 * n)()
        self._check(self._lib.laserkv_profile_end(self._ctx, ms, cnt))
        return {KERNEL_NAMES[i]: (float(ms[i]), int(cnt[i])) for i in range(n)}

    def laserkv_profile_isolate(self, kernel):
        """kernel: a name from KERNEL_NAMES, or None to launch every kernel again."""
        self._check(self._lib.laserkv_profile_isolate(self._ctx, -1 if kernel is None else KERNEL_NAMES.index(kernel)))

    def laserkv_layer_plan(self, n_tok, s_block, w, B, n, alpha, lse_complete=False):
        """How laserkv_compress_layer cuts up a layer of these sizes: {name of LAYER_PLAN: value}."""
        plan = (C.c_int64 * len(LAYER_PLAN))()
        rc = self._lib.laserkv_layer_plan(self._ctx, n_tok, s_block, w, B, n, alpha, 1 if lse_complete else 0, plan)
        if rc != LKV_OK:
            raise LaserKVError(rc, "layer_plan: null, or sizes that compress_layer refuses")
        return dict(zip(LAYER_PLAN, map(int, plan)))
