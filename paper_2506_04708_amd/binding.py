"""Thin ctypes binding of libstand.so (see include/stand.h): argument marshalling only.

Device buffers are torch tensors (PyTorch-ROCm is used for memory and streams, nothing else);
every step of the path runs in the HIP kernels of the library.  There is no CPU fallback: if
the library has not been built, importing this module raises.
"""
import ctypes as C
import os

import numpy as np
import torch

_HERE = os.path.dirname(os.path.abspath(__file__))
LIB_PATH = os.path.join(_HERE, "libstand.so")

STAND_BF16, STAND_F32 = 0, 1
DRAFT_GUMBEL_TOPK, DRAFT_MULTINOMIAL, DRAFT_DETERMINISTIC = 0, 1, 2
MERGE_MEAN, MERGE_REPLACE = 0, 1
STEP_AUTO, STEP_SERIAL, STEP_FUSED = 0, 1, 2
MAX_ORDER = 8

EXPORTED = [
    "stand_create", "stand_destroy", "stand_depth", "stand_set_context", "stand_reorder", "stand_update",
    "stand_draft", "stand_verify", "stand_step", "stand_row_results", "stand_table_export", "stand_table_import",
    "stand_get_context", "stand_get_stats", "stand_strerror", "stand_last_hip_error",
    "stand_profile_begin", "stand_profile_end", "stand_copy_bytes", "stand_read_rows", "stand_set_filter_margin",
    "stand_tree_initial", "stand_tree_select", "stand_get_node_counts", "stand_reset_node_counts",
    "stand_tree_packing", "stand_verify_static", "stand_static_scratch_need",
    "stand_set_step_plan", "stand_set_wait_limit", "stand_step_timeline", "stand_step_is_one_launch",
    "stand_get_record_slots",
]


class Config(C.Structure):
    _fields_ = [
        ("vocab", C.c_int32), ("max_batch", C.c_int32), ("order_min", C.c_int32), ("order_max", C.c_int32),
        ("topk", C.c_int32), ("tree_nodes", C.c_int32), ("tree_parent", C.POINTER(C.c_int32)),
        ("temperature", C.c_float), ("table_capacity", C.c_uint64), ("max_probe", C.c_int32),
        ("seed", C.c_uint64), ("logits_dtype", C.c_int32), ("update_mode", C.c_int32), ("device", C.c_int32),
        ("draft_mode", C.c_int32), ("merge_policy", C.c_int32),
    ]


class Stats(C.Structure):
    _fields_ = [
        ("hits", C.c_uint64 * (MAX_ORDER + 1)), ("misses", C.c_uint64),
        ("inserts", C.c_uint64), ("merges", C.c_uint64), ("drops", C.c_uint64),
        ("near_threshold", C.c_uint64), ("tokens_emitted", C.c_uint64), ("accept_tests", C.c_uint64),
        ("filter_mismatch", C.c_uint64), ("wait_expired", C.c_uint64), ("late_paths", C.c_uint64),
    ]


def load_library():
    if not os.path.exists(LIB_PATH):
        raise ImportError("libstand.so is not built: run `python -c 'import __graft_entry__ as g; g.build()'` "
                          "(or python -m paper_2506_04708_amd.build) first; there is no fallback path")
    lib = C.CDLL(LIB_PATH)
    vp, i32p = C.c_void_p, C.c_void_p
    lib.stand_create.argtypes = [C.POINTER(Config), C.POINTER(vp)]
    lib.stand_destroy.argtypes = [vp]
    lib.stand_depth.argtypes = [vp]
    lib.stand_set_context.argtypes = [vp, C.c_int32, i32p, C.c_int32, vp]
    lib.stand_reorder.argtypes = [vp, i32p, vp]
    lib.stand_update.argtypes = [vp, C.c_uint64, vp, i32p, i32p, i32p, vp]
    lib.stand_draft.argtypes = [vp, C.c_uint64, i32p, vp]
    lib.stand_verify.argtypes = [vp, C.c_uint64, vp, i32p, i32p, i32p, vp]
    lib.stand_verify_static.argtypes = [vp, C.c_uint64, vp, i32p, i32p, i32p, vp]
    lib.stand_static_scratch_need.argtypes = [vp]
    lib.stand_static_scratch_need.restype = C.c_uint64
    lib.stand_set_step_plan.argtypes = [vp, C.c_int32, C.c_int32, C.c_int32, C.c_int32, C.c_uint32]
    lib.stand_set_wait_limit.argtypes = [vp, C.c_uint64]
    lib.stand_step_is_one_launch.argtypes = [vp]
    lib.stand_step_timeline.argtypes = [vp, C.c_int32, vp, C.POINTER(C.c_uint64)]
    lib.stand_step.argtypes = [vp, C.c_uint64, vp, i32p, i32p, i32p, i32p, i32p, vp]
    lib.stand_row_results.argtypes = [vp, vp, vp, vp, vp, vp]
    lib.stand_table_export.argtypes = [vp, vp, C.POINTER(C.c_uint64)]
    lib.stand_table_import.argtypes = [vp, vp, C.c_uint64]
    lib.stand_get_context.argtypes = [vp, C.c_int32, i32p, C.c_int32, C.POINTER(C.c_int64), vp]
    lib.stand_get_stats.argtypes = [vp, C.POINTER(Stats)]
    lib.stand_set_filter_margin.argtypes = [vp, C.c_float]
    lib.stand_profile_begin.argtypes = [vp, C.c_int32]
    lib.stand_profile_end.argtypes = [vp, C.POINTER(C.c_double), C.POINTER(C.c_int32)]
    lib.stand_copy_bytes.argtypes = [vp, vp, C.c_uint64, vp]
    lib.stand_read_rows.argtypes = [vp, C.c_uint64, C.c_uint64, vp, vp]
    lib.stand_tree_initial.argtypes = [C.c_int32, i32p, C.c_int32, C.POINTER(C.c_int32)]
    lib.stand_tree_select.argtypes = [i32p, vp, C.c_int32, C.c_int32, i32p, i32p]
    lib.stand_get_node_counts.argtypes = [vp, vp]
    lib.stand_get_record_slots.argtypes = [vp, vp]
    lib.stand_tree_packing.argtypes = [vp, vp, vp, vp]
    lib.stand_reset_node_counts.argtypes = [vp]
    lib.stand_strerror.restype = C.c_char_p
    lib.stand_strerror.argtypes = [C.c_int]
    lib.stand_last_hip_error.argtypes = [vp]
    return lib


_lib = None


def copy_bytes(dst, src, nbytes, stream=None):
    """Plain device copy (measurement aid): dst, src are torch tensors on the GPU."""
    rc = lib().stand_copy_bytes(dst.data_ptr(), src.data_ptr(), nbytes, stream)
    if rc:
        raise RuntimeError("stand_copy_bytes: %s" % lib().stand_strerror(rc).decode())


def read_rows(src, row_bytes, rows, sink, stream=None):
    """Bare read of `rows` rows in the row pass's launch shape (measurement aid); sink: int32 tensor of 4 * rows."""
    rc = lib().stand_read_rows(src.data_ptr(), row_bytes, rows, sink.data_ptr(), stream)
    if rc:
        raise RuntimeError("stand_read_rows: %s" % lib().stand_strerror(rc).decode())


def tree_initial(levels=20):
    """parent[] of the initial tree of the tree optimisation (host only)."""
    n = C.c_int32(0)
    rc = lib().stand_tree_initial(levels, None, 0, C.byref(n))
    if rc:
        raise RuntimeError("stand_tree_initial: %s" % lib().stand_strerror(rc).decode())
    out = np.zeros(n.value, np.int32)
    rc = lib().stand_tree_initial(levels, out.ctypes.data, n.value, C.byref(n))
    if rc:
        raise RuntimeError("stand_tree_initial: %s" % lib().stand_strerror(rc).decode())
    return out


def tree_select(parent, counts, n_keep):
    """(new parent[], old ids) of the n_keep most often accepted nodes, re-packed (host only)."""
    parent = np.ascontiguousarray(parent, np.int32)
    counts = np.ascontiguousarray(counts, np.uint64)
    out = np.zeros(n_keep, np.int32)
    old = np.zeros(n_keep, np.int32)
    rc = lib().stand_tree_select(parent.ctypes.data, counts.ctypes.data, parent.shape[0], n_keep, out.ctypes.data,
                                 old.ctypes.data)
    if rc:
        raise RuntimeError("stand_tree_select: %s" % lib().stand_strerror(rc).decode())
    return out, old


def lib():
    global _lib
    if _lib is None:
        _lib = load_library()
    return _lib


class StandError(RuntimeError):
    pass


def _check(rc, handle=None):
    if rc:
        msg = lib().stand_strerror(rc).decode()
        if handle is not None and rc == -3:
            msg += " [hip error %d]" % lib().stand_last_hip_error(handle)
        raise StandError("libstand: %s (%d)" % (msg, rc))


def _dptr(t, dtype=None):
    # (a plain integer: the functions' argtypes make the pointer)
    if t is None:
        return None
    assert t.is_cuda and t.is_contiguous()
    if dtype is not None:
        assert t.dtype is dtype, (t.dtype, dtype)
    return t.data_ptr()


def _stream_ptr():
    return torch.cuda.current_stream().cuda_stream


# The same for calls that have just been given tensors of the GPU (torch's runtime is up): without the stream object, which
# costs more than the rest of such a call's arguments together.
try:
    _raw_stream, _device = torch._C._cuda_getCurrentRawStream, torch._C._cuda_getDevice

    def _stream_ptr_up():
        return _raw_stream(_device())
except AttributeError:   # (a torch without them)
    _stream_ptr_up = _stream_ptr


class Stand:
    """One n-gram table shared by B trajectories on one GPU; methods carry the C ABI's names."""

    def __init__(self, vocab, max_batch, order_min, order_max, topk, tree_parent, temperature, table_capacity,
                 max_probe, seed, logits_dtype, device=0, draft_mode=0, update_mode=0, merge_policy=0):
        par = np.ascontiguousarray(tree_parent, dtype=np.int32)
        cfg = Config(vocab, max_batch, order_min, order_max, topk, par.shape[0],
                     par.ctypes.data_as(C.POINTER(C.c_int32)), temperature, table_capacity, max_probe, seed,
                     logits_dtype, update_mode, device, draft_mode, merge_policy)
        self.h = C.c_void_p()
        _check(lib().stand_create(C.byref(cfg), C.byref(self.h)))
        self.B, self.N, self.K, self.V = max_batch, par.shape[0], topk, vocab
        self._lib, self._logits = lib(), max_batch * par.shape[0] * vocab
        self.D = lib().stand_depth(self.h)
        self.W = self.D + 1
        self.logits_dtype = logits_dtype
        self.device = torch.device("cuda", device)

    def close(self):
        if getattr(self, "h", None):
            lib().stand_destroy(self.h)
            self.h = None

    def __del__(self):
        try:
            self.close()
        except Exception:
            pass

    def _logits_ptr(self, logits):
        assert logits.is_cuda and logits.is_contiguous() and logits.numel() == self._logits
        if self.logits_dtype == STAND_BF16:
            assert logits.dtype in (torch.bfloat16, torch.uint16, torch.int16)
        else:
            assert logits.dtype == torch.float32
        return logits.data_ptr()

    def new_outputs(self):
        i32 = dict(dtype=torch.int32, device=self.device)
        return (torch.empty((self.B, self.W), **i32), torch.empty((self.B, self.W), **i32),
                torch.empty((self.B,), **i32), torch.empty((self.B, self.N), **i32))

    def set_context(self, b, tokens):
        t = np.ascontiguousarray(tokens, dtype=np.int32)
        _check(lib().stand_set_context(self.h, b, t.ctypes.data_as(C.c_void_p), t.shape[0], _stream_ptr()), self.h)

    def reorder(self, src_of):
        s = np.ascontiguousarray(src_of, dtype=np.int32)
        assert s.shape[0] == self.B
        _check(lib().stand_reorder(self.h, s.ctypes.data_as(C.c_void_p), _stream_ptr()), self.h)

    def update(self, step, logits, commit_tok, commit_row, commit_len):
        assert commit_tok.shape == (self.B, self.W) and commit_row.shape == (self.B, self.W) and commit_len.shape == (self.B,)
        _check(self._lib.stand_update(self.h, step, self._logits_ptr(logits), _dptr(commit_tok, torch.int32),
                                  _dptr(commit_row, torch.int32), _dptr(commit_len, torch.int32), _stream_ptr_up()), self.h)

    def draft(self, step, draft_tok):
        assert draft_tok.shape == (self.B, self.N)
        _check(self._lib.stand_draft(self.h, step, _dptr(draft_tok, torch.int32), _stream_ptr_up()), self.h)

    def verify(self, step, logits, out_tok, out_node, out_len):
        _check(self._lib.stand_verify(self.h, step, self._logits_ptr(logits), _dptr(out_tok, torch.int32),
                                  _dptr(out_node, torch.int32), _dptr(out_len, torch.int32), _stream_ptr_up()), self.h)

    def verify_static(self, step, logits, out_tok, out_node, out_len):
        _check(self._lib.stand_verify_static(self.h, step, self._logits_ptr(logits), _dptr(out_tok, torch.int32),
                                         _dptr(out_node, torch.int32), _dptr(out_len, torch.int32), _stream_ptr_up()), self.h)

    def static_scratch_need(self):
        return int(lib().stand_static_scratch_need(self.h))

    def step(self, step, logits, out_tok, out_node, out_len, next_draft_tok, force_tok=None):
        _check(self._lib.stand_step(self.h, step, self._logits_ptr(logits), _dptr(out_tok, torch.int32),
                                _dptr(out_node, torch.int32), _dptr(out_len, torch.int32),
                                _dptr(next_draft_tok, torch.int32), _dptr(force_tok, torch.int32), _stream_ptr_up()), self.h)

    def row_results(self):
        rows = self.B * self.N
        m = torch.empty(rows, dtype=torch.float32, device=self.device)
        s = torch.empty(rows, dtype=torch.float32, device=self.device)
        idx = torch.empty((rows, self.K), dtype=torch.int32, device=self.device)
        p = torch.empty((rows, self.K), dtype=torch.float32, device=self.device)
        _check(self._lib.stand_row_results(self.h, _dptr(m), _dptr(s), _dptr(idx), _dptr(p), _stream_ptr_up()), self.h)
        return m, s, idx, p

    def table_export(self):
        n = C.c_uint64(0)
        _check(lib().stand_table_export(self.h, None, C.byref(n)), self.h)
        buf = np.zeros(max(int(n.value), 1), np.uint8)
        n2 = C.c_uint64(buf.shape[0])
        _check(lib().stand_table_export(self.h, buf.ctypes.data_as(C.c_void_p), C.byref(n2)), self.h)
        return buf[: int(n2.value)]

    def table_import(self, buf):
        b = np.ascontiguousarray(buf, dtype=np.uint8)
        _check(lib().stand_table_import(self.h, b.ctypes.data_as(C.c_void_p), b.shape[0]), self.h)

    def get_context(self, b, n):
        out = np.zeros(max(n, 1), np.int32)
        ln = C.c_int64(0)
        _check(lib().stand_get_context(self.h, b, out.ctypes.data_as(C.c_void_p), n, C.byref(ln), _stream_ptr()), self.h)
        return out[:n], int(ln.value)

    def set_step_plan(self, mode=0, upper_depth=2, tail_groups=0, shuffle=0, rows_first=0):
        _check(lib().stand_set_step_plan(self.h, mode, upper_depth, tail_groups, rows_first, shuffle), self.h)

    def step_is_one_launch(self):
        return lib().stand_step_is_one_launch(self.h) == 1

    def set_wait_limit(self, microseconds):
        _check(lib().stand_set_wait_limit(self.h, microseconds), self.h)

    def step_timeline(self, enable=True, read=False):
        """Switches the recording of the one-launch step's clock readings on or off; with read=True returns
        (row_start, row_end, per-trajectory stamps [B, 8]) of the last such step in microseconds from row_start."""
        rate = C.c_uint64(0)
        buf = np.zeros(2 + 8 * self.B, np.uint64) if read else None
        _check(lib().stand_step_timeline(self.h, int(enable), buf.ctypes.data if read else None, C.byref(rate)), self.h)
        if not read:
            return None
        us = (buf.astype(np.int64) - np.int64(buf[0])) * (1e6 / rate.value)
        return float(us[0]), float(us[1]), us[2:].reshape(self.B, 8)

    def set_filter_margin(self, margin):
        _check(lib().stand_set_filter_margin(self.h, margin), self.h)

    def profile_begin(self, max_launches):
        _check(lib().stand_profile_begin(self.h, max_launches), self.h)

    def profile_end(self):
        ms = C.c_double(0)
        n = C.c_int32(0)
        _check(lib().stand_profile_end(self.h, C.byref(ms), C.byref(n)), self.h)
        return ms.value, n.value

    def stats(self):
        s = Stats()
        _check(lib().stand_get_stats(self.h, C.byref(s)), self.h)
        return s

    def tree_packing(self):
        """(mask [B, N, N] uint8, positions [B, N] int64) of the pending drafts, on the GPU."""
        mask = torch.empty((self.B, self.N, self.N), dtype=torch.uint8, device=self.device)
        pos = torch.empty((self.B, self.N), dtype=torch.int64, device=self.device)
        _check(self._lib.stand_tree_packing(self.h, _dptr(mask), _dptr(pos), _stream_ptr_up()), self.h)
        return mask, pos

    def record_slots(self, rows_per_trajectory, orders):
        """Slot of every merge record of the last update, [B, R, orders] (-1: no such record, or dropped)."""
        out = np.zeros(self.B * rows_per_trajectory * orders, np.int64)
        _check(lib().stand_get_record_slots(self.h, out.ctypes.data), self.h)
        return out.reshape(self.B, rows_per_trajectory, orders)

    def node_counts(self):
        out = np.zeros(self.N, np.uint64)
        _check(lib().stand_get_node_counts(self.h, out.ctypes.data), self.h)
        return out

    def reset_node_counts(self):
        _check(lib().stand_reset_node_counts(self.h), self.h)
