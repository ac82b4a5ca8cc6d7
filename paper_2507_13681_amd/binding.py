"""Thin binding of libloopserve (see include/loopserve.h, include/loopserve_test_hooks.h).

Argument marshalling only (natively, by csrc/ls_py.c, for the calls of a serving loop; through ctypes for
the rest): every step of the path runs in the HIP kernels of the library.  PyTorch supplies device memory and
the current stream.  The library must have been built
(`python -m paper_2507_13681_amd.build` or `__graft_entry__.build()`); loading fails loudly
otherwise -- there is no CPU fallback.
"""
from __future__ import annotations

import ctypes as C
import math
import os

import torch

_DIR = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_DIR, "libloopserve.so")
LS_BF16, LS_F32 = 0, 1
LS_MAX_N, LS_MAX_W = 262144, 256
_lib = None

ENTRY_POINTS = ("ls_workspace_bytes", "ls_create", "ls_destroy", "ls_last_error",
                "ls_score", "ls_select", "ls_sparse_prefill", "ls_kv_compress", "ls_poll_status")
# bits of the device status word (ls_poll_status)
LS_STAT_WALK_TIMEOUT, LS_STAT_S_TRUNCATED, LS_STAT_V_TRUNCATED, LS_STAT_S_RANGE, LS_STAT_V_INVALID = 1, 2, 4, 8, 16
LS_STAT_MERGE_RANGE = 32


class LsShape(C.Structure):
    _fields_ = [("B", C.c_int32), ("Hq", C.c_int32), ("Hkv", C.c_int32), ("d", C.c_int32),
                ("n", C.c_int64), ("n_hat", C.c_int64), ("w", C.c_int32), ("dtype", C.c_int32),
                ("scale", C.c_float)]


class LoopServeError(RuntimeError):
    pass


def load_library():
    """dlopen the HIP library and declare the signatures of include/loopserve.h."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(LIB_PATH):
        raise LoopServeError(f"{LIB_PATH} is missing: build it with `python -m paper_2507_13681_amd.build`")
    lib = C.CDLL(LIB_PATH)
    vp, i32, i64, f32 = C.c_void_p, C.c_int32, C.c_int64, C.c_float
    sp = C.POINTER(LsShape)
    lib.ls_workspace_bytes.restype = C.c_size_t
    lib.ls_workspace_bytes.argtypes = [sp, i32]
    lib.ls_create.restype = C.c_int
    lib.ls_create.argtypes = [C.POINTER(vp), C.c_int, C.c_size_t]
    lib.ls_destroy.restype = None
    lib.ls_destroy.argtypes = [vp]
    lib.ls_last_error.restype = C.c_char_p
    lib.ls_last_error.argtypes = [vp]
    lib.ls_score.restype = C.c_int
    lib.ls_score.argtypes = [vp, sp, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.ls_select.restype = C.c_int
    lib.ls_select.argtypes = [vp, sp, f32, vp, vp, vp, vp, vp, vp, vp, i32, vp, vp, i32, vp, vp]
    lib.ls_score_window.restype = C.c_int
    lib.ls_score_window.argtypes = [vp, sp, vp, vp, vp, vp, vp]
    lib.ls_select_exact.restype = C.c_int
    lib.ls_select_exact.argtypes = [vp, sp, f32, vp, vp, vp, vp, vp, vp, vp, i32, vp, vp, i32, vp, vp]
    lib.ls_merge_lines.restype = C.c_int
    lib.ls_merge_lines.argtypes = [vp, sp] + [vp, vp, i32] * 6 + [vp]
    lib.ls_sparse_prefill.restype = C.c_int
    lib.ls_sparse_prefill.argtypes = [vp, sp, vp, vp, vp, vp, vp, i32, vp, vp, i32, vp, vp, vp]
    lib.ls_kv_compress.restype = C.c_int
    lib.ls_kv_compress.argtypes = [vp, sp, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.ls_kv_compress_static.restype = C.c_int
    lib.ls_kv_compress_static.argtypes = [C.c_int, sp, i32, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.ls_static_scratch_bytes.restype = C.c_size_t
    lib.ls_static_scratch_bytes.argtypes = []
    lib.ls_decode_attend.restype = C.c_int
    lib.ls_decode_attend.argtypes = [vp, sp, i32, i32, vp, vp, vp, vp, vp, vp, vp, vp, vp]
    lib.ls_decode_workspace_bytes.restype = C.c_size_t
    lib.ls_decode_workspace_bytes.argtypes = [sp, i32, i32]
    lib.ls_debug_copy_compress_score.restype = C.c_int
    lib.ls_debug_copy_compress_score.argtypes = [vp, sp, vp, vp]
    lib.ls_poll_status.restype = C.c_int
    lib.ls_poll_status.argtypes = [vp, C.POINTER(i32), vp]
    lib.ls_debug_set_walk_spin_limit.restype = C.c_int
    lib.ls_debug_set_walk_spin_limit.argtypes = [vp, i32]
    lib.ls_debug_set_counters.restype = C.c_int
    lib.ls_debug_set_counters.argtypes = [vp, i32, vp]
    lib.ls_debug_fill_workspace.restype = C.c_int
    lib.ls_debug_fill_workspace.argtypes = [vp, i32, vp]
    lib.ls_debug_copy_select_order.restype = C.c_int
    lib.ls_debug_copy_select_order.argtypes = [vp, sp, vp, vp, vp, vp]
    lib.ls_debug_prefill_in_pieces.restype = C.c_int
    lib.ls_debug_prefill_in_pieces.argtypes = [sp]
    lib.ls_debug_score_route.restype = C.c_int
    lib.ls_debug_score_route.argtypes = [sp, i32, i32, C.POINTER(i32), C.POINTER(i64)]
    lib.ls_debug_copy_prefill_queues.restype = C.c_int
    lib.ls_debug_copy_prefill_queues.argtypes = [vp, sp, vp, vp, C.POINTER(i32), C.POINTER(i32), vp]
    lib.ls_profile_enable.restype = C.c_int
    lib.ls_profile_enable.argtypes = [vp, C.c_int]
    lib.ls_profile_prefill_kernel_ms.restype = C.c_int
    lib.ls_profile_prefill_kernel_ms.argtypes = [vp, C.POINTER(C.c_double), C.POINTER(i32)]
    _lib = lib
    return lib


def _load_native():
    """The CPython module over the C ABI, built beside the library."""
    try:
        from . import _lsnative
    except ImportError as e:
        raise LoopServeError(f"_lsnative.so cannot be loaded ({e}): build it with `python -m paper_2507_13681_amd.build`") from e
    return _lsnative


def make_shape(B, Hq, Hkv, d, n, n_hat, w, dtype, scale=0.0) -> LsShape:
    code = {torch.bfloat16: LS_BF16, torch.float32: LS_F32, "bf16": LS_BF16, "f32": LS_F32}[dtype]
    return LsShape(B, Hq, Hkv, d, n, n_hat, w, code, float(scale))


def workspace_bytes(shape: LsShape, budget: int = 0) -> int:
    return int(load_library().ls_workspace_bytes(C.byref(shape), budget))


def decode_workspace_bytes(shape: LsShape, cap: int, T: int) -> int:
    return int(load_library().ls_decode_workspace_bytes(C.byref(shape), cap, T))


def _ptr(t):
    if t is None:
        return None
    assert t.is_cuda and t.is_contiguous(), "tensors must be contiguous device tensors"
    return C.c_void_p(t.data_ptr())


def _stream():
    return C.c_void_p(torch._C._cuda_getCurrentRawStream(torch._C._cuda_getDevice()))


class Context:
    """An ls_ctx: a device workspace that the four calls carve their scratch from."""

    def __init__(self, shape: LsShape | None = None, budget: int = 0, device: int = 0, workspace: int | None = None):
        self.lib = load_library()
        self.native = _load_native()
        if workspace is None:
            workspace = workspace_bytes(shape, budget)
            if workspace == 0:
                raise LoopServeError("invalid shape")
        self.workspace = int(workspace)
        self.device = device
        h = C.c_void_p()
        rc = self.lib.ls_create(C.byref(h), device, self.workspace)
        if rc != 0:
            raise LoopServeError(f"ls_create failed with {rc}")
        self.h = h
        self.hv = h.value                        # what the native marshalling takes; 0 (an error in every call) once closed

    def close(self):
        if getattr(self, "h", None):
            self.lib.ls_destroy(self.h)
            self.h = None
            self.hv = 0

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _check(self, rc):
        if rc != 0:
            raise LoopServeError(f"{self.lib.ls_last_error(self.h).decode()} (status {rc})")

    # -- the entry points, same names as the C ABI (the marshalling is native: csrc/ls_py.c) ------------
    def ls_score(self, shape, q_win, k, vert, slash, vmax, smax, total, q_pos=None):
        rc = self.native.score(self.hv, shape, q_win, q_pos, k, vert, slash, vmax, smax, total)
        if rc:
            self._check(rc)

    def ls_select(self, shape, alpha, vert, slash, vmax, smax, total, v_idx, v_cnt, s_idx, s_cnt, accounted=None):
        rc = self.native.select_lines(self.hv, shape, alpha, vert, slash, vmax, smax, total, v_idx, v_cnt, s_idx, s_cnt, accounted)
        if rc:
            self._check(rc)

    def ls_score_window(self, shape, q_win, k, a_win, q_pos=None):
        rc = self.native.score_window(self.hv, shape, q_win, q_pos, k, a_win)
        if rc:
            self._check(rc)

    def ls_select_exact(self, shape, alpha, a_win, vert, slash, total, v_idx, v_cnt, s_idx, s_cnt, accounted=None, q_pos=None):
        rc = self.native.select_exact(self.hv, shape, alpha, a_win, q_pos, vert, slash, total, v_idx, v_cnt, s_idx, s_cnt, accounted)
        if rc:
            self._check(rc)

    def ls_merge_lines(self, shape, a, b, out):
        """a, b, out: dicts with v_idx, v_cnt, s_idx, s_cnt (as alloc_select returns them)."""
        rc = self.native.merge_lines(self.hv, shape, a["v_idx"], a["v_cnt"], a["s_idx"], a["s_cnt"],
                                     b["v_idx"], b["v_cnt"], b["s_idx"], b["s_cnt"],
                                     out["v_idx"], out["v_cnt"], out["s_idx"], out["s_cnt"])
        if rc:
            self._check(rc)

    def ls_sparse_prefill(self, shape, q, k, v, v_idx, v_cnt, s_idx, s_cnt, out, lse=None):
        rc = self.native.sparse_prefill(self.hv, shape, q, k, v, v_idx, v_cnt, s_idx, s_cnt, out, lse)
        if rc:
            self._check(rc)

    def ls_kv_compress(self, shape, budget, q_obs, k, v, keep_idx, keep_cnt, k_out=None, v_out=None):
        rc = self.native.kv_compress(self.hv, shape, budget, q_obs, k, v, keep_idx, keep_cnt, k_out, v_out)
        if rc:
            self._check(rc)

    def ls_decode_attend(self, shape, q, k_c, v_c, cnt, k_t, v_t, out, lse=None):
        rc = self.native.decode_attend(self.hv, shape, q, k_c, v_c, cnt, k_t, v_t, out, lse)
        if rc:
            self._check(rc)

    def ls_poll_status(self) -> int:
        """Waits for the current stream, returns the context's device status word and clears it."""
        word = C.c_int32()
        self._check(self.lib.ls_poll_status(self.h, C.byref(word), _stream()))
        return word.value

    def debug_set_walk_spin_limit(self, limit: int):
        self._check(self.lib.ls_debug_set_walk_spin_limit(self.h, limit))

    def debug_set_counters(self, value: int):
        self._check(self.lib.ls_debug_set_counters(self.h, value, _stream()))

    def debug_fill_workspace(self, value: int):
        self._check(self.lib.ls_debug_fill_workspace(self.h, value, _stream()))

    def debug_select_order(self, shape):
        """Of the last ls_select call: ranges a list (0: none are left out), how many were left out to the end [2][heads], how many of heads that were walked again."""
        import numpy as np
        heads = shape.B * shape.Hq
        left, again, ranges = np.zeros((2, heads), np.int32), np.zeros(heads, np.int32), C.c_int32()
        self._check(self.lib.ls_debug_copy_select_order(self.h, C.byref(shape), left.ctypes.data_as(C.c_void_p), again.ctypes.data_as(C.c_void_p), C.byref(ranges), _stream()))
        return ranges.value, left, again

    def debug_prefill_queues(self, shape):
        """Items of the last ls_sparse_prefill call by XCD (eight int arrays of item words), row blocks a head, cuts through items."""
        import numpy as np
        items = shape.B * shape.Hq * ((int(shape.n) + 127) // 128 + 1)        # at least B * Hq * nqb
        qlen = np.zeros(8, dtype=np.int32)
        nqb, cuts = C.c_int32(), C.c_int32()
        # the library packs the queues at the true stride B * Hq * nqb: read flat, then cut
        flat = np.zeros(8 * items, dtype=np.uint32)
        self._check(self.lib.ls_debug_copy_prefill_queues(self.h, C.byref(shape), flat.ctypes.data_as(C.c_void_p),
                                                          qlen.ctypes.data_as(C.c_void_p), C.byref(nqb), C.byref(cuts), _stream()))
        stride = shape.B * shape.Hq * nqb.value
        return [flat[x * stride: x * stride + int(qlen[x])].copy() for x in range(8)], nqb.value, cuts.value

    def profile_enable(self, on=True):
        self._check(self.lib.ls_profile_enable(self.h, 1 if on else 0))

    def profile_prefill_kernel_ms(self):
        ms, cnt = C.c_double(), C.c_int32()
        self._check(self.lib.ls_profile_prefill_kernel_ms(self.h, C.byref(ms), C.byref(cnt)))
        return ms.value, cnt.value

    def debug_compress_score(self, shape, dst):
        self._check(self.lib.ls_debug_copy_compress_score(self.h, C.byref(shape), _ptr(dst), _stream()))


def ls_kv_compress_static(shape, budget, q_obs, k, v, keep_idx, keep_cnt, k_out=None, v_out=None, device=0):
    """ls_kv_compress without a context, on the library's static scratch (allocates nothing)."""
    lib = load_library()
    rc = lib.ls_kv_compress_static(device, C.byref(shape), budget, _ptr(q_obs), _ptr(k), _ptr(v), _ptr(keep_idx),
                                   _ptr(keep_cnt), _ptr(k_out), _ptr(v_out), _stream())
    if rc != 0:
        raise LoopServeError(f"{lib.ls_last_error(None).decode()} (status {rc})")


def static_scratch_bytes() -> int:
    return int(load_library().ls_static_scratch_bytes())


# -- convenience: allocate outputs with torch and run one call ----------------------------------

def score_route(shape: LsShape, mode: int, positions: bool = False) -> dict:
    """Which scoring kernels a call of this shape takes (test hook, no GPU needed); mode: 0 ls_score of the newest rows, 1 ls_score
    otherwise, 2 ls_kv_compress, 3 ls_score_window; positions: explicit ones.  `begins`: where the ranges of the statistics pass begin, and n."""
    lib, words = load_library(), (C.c_int32 * 9)()
    rc = lib.ls_debug_score_route(C.byref(shape), mode, int(positions), words, None)
    if rc != 0:
        raise LoopServeError(f"ls_debug_score_route failed with {rc}")
    begins = (C.c_int64 * (words[0] + 1))()
    lib.ls_debug_score_route(C.byref(shape), mode, int(positions), words, begins)
    return dict(ranges=words[0], chunks=words[1], shares=words[2], folds=bool(words[3]), joins=bool(words[4]), streams=bool(words[5]),
                band_heads=words[6], band_rows=words[7], band_shares=words[8], begins=list(begins))


def prefill_in_pieces(shape: LsShape) -> bool:
    """Whether ls_sparse_prefill shares the work of such a turn out in pieces, not by work queues (test hook, no GPU needed)."""
    rc = load_library().ls_debug_prefill_in_pieces(C.byref(shape))
    if rc < 0:
        raise LoopServeError(f"ls_debug_prefill_in_pieces failed with {rc}")
    return rc == 1


def alloc_score(shape: LsShape, device="cuda"):
    B, Hq, n = shape.B, shape.Hq, shape.n
    f = dict(dtype=torch.float32, device=device)
    return dict(vert=torch.empty(B, Hq, n, **f), slash=torch.empty(B, Hq, n, **f), vmax=torch.empty(B, Hq, n, **f),
                smax=torch.empty(B, Hq, n, **f), total=torch.empty(B, Hq, **f))


def alloc_select(shape: LsShape, cap_v=None, cap_s=None, device="cuda", accounted=True):
    B, Hq, n = shape.B, shape.Hq, shape.n
    i = dict(dtype=torch.int32, device=device)
    return dict(v_idx=torch.empty(B, Hq, cap_v or n, **i), v_cnt=torch.empty(B, Hq, **i),
                s_idx=torch.empty(B, Hq, cap_s or n, **i), s_cnt=torch.empty(B, Hq, **i),
                accounted=torch.empty(B, Hq, dtype=torch.float32, device=device) if accounted else None)


def default_scale(d):
    return 1.0 / math.sqrt(d)
