"""ctypes binding of include/dfa.h.  Argument marshalling only."""
from __future__ import annotations

import collections
import ctypes
import functools
import os

import torch

_PKG_DIR = os.path.dirname(os.path.abspath(__file__))
_LIB_PATH = os.path.join(_PKG_DIR, "libdfa.so")
_lib = None

DFA_BF16, DFA_F32 = 0, 1
DFA_ERR_NULL = -1
DFA_STEP_IDLE, DFA_STEP_DIAG, DFA_STEP_OWN, DFA_STEP_HELP = 0, 1, 2, 3
STEP_NAMES = {0: "idle", 1: "diag", 2: "own", 3: "help"}
# a call takes rows * row stride (elements) of one head's slice up to this (include/dfa.h: 32-bit byte offsets)
MAX_SLICE = (1 << 29) - 1


class DfaError(RuntimeError):
    def __init__(self, status: int, where: str):
        self.status = status
        super().__init__(f"{where}: {dfa_status_str(status)} ({status})")


class DfaShape(ctypes.Structure):
    _fields_ = [
        ("h_q", ctypes.c_int32), ("h_kv", ctypes.c_int32),
        ("s_q", ctypes.c_int32), ("s_k", ctypes.c_int32),
        ("d", ctypes.c_int32), ("dtype", ctypes.c_int32), ("o_dtype", ctypes.c_int32),
        ("causal", ctypes.c_int32), ("scale", ctypes.c_float), ("reserved", ctypes.c_int32),
        ("q_stride_h", ctypes.c_int64), ("q_stride_s", ctypes.c_int64),
        ("kv_stride_h", ctypes.c_int64), ("kv_stride_s", ctypes.c_int64),
        ("o_stride_h", ctypes.c_int64), ("o_stride_s", ctypes.c_int64),
        ("lse_stride_h", ctypes.c_int64),
        ("dq_stride_h", ctypes.c_int64), ("dq_stride_s", ctypes.c_int64),
        ("dkv_stride_h", ctypes.c_int64), ("dkv_stride_s", ctypes.c_int64),
    ]


class DfaMergeDesc(ctypes.Structure):
    _fields_ = [("heads", ctypes.c_int32), ("rows", ctypes.c_int32), ("d", ctypes.c_int32),
                ("o_dtype", ctypes.c_int32),
                ("a_stride_h", ctypes.c_int64), ("a_stride_s", ctypes.c_int64), ("lse_a_stride_h", ctypes.c_int64),
                ("b_stride_h", ctypes.c_int64), ("b_stride_s", ctypes.c_int64), ("lse_b_stride_h", ctypes.c_int64)]


class DfaFwdPair(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("q", "k", "v", "o", "lse")] + [
        (n, ctypes.c_int64) for n in ("o_stride_h", "o_stride_s", "lse_stride_h")] + [
        ("accumulate", ctypes.c_int32), ("reserved", ctypes.c_int32)]


class DfaMergePair(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("o_a", "lse_a", "o_b", "lse_b")]


class DfaFwdSpan(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("q", "k", "v", "o", "lse")] + [
        (n, ctypes.c_int64) for n in ("o_stride_h", "o_stride_s", "lse_stride_h")] + [
        (n, ctypes.c_int32) for n in ("n_keys", "own", "accumulate", "reserved")]


class DfaForm(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int32) for n in ("rows", "parts", "cuts", "q_cuts")]


class DfaBwdPair(ctypes.Structure):
    _fields_ = [(n, ctypes.c_void_p) for n in ("q", "k", "v", "lse", "delta", "dO", "dq", "dk", "dv")] + [
        ("accumulate_dq", ctypes.c_int32), ("accumulate_dkv", ctypes.c_int32)]


class DfaStep(ctypes.Structure):
    _fields_ = [("t", ctypes.c_int32), ("kind", ctypes.c_int32), ("q_chunk", ctypes.c_int32),
                ("kv_chunk", ctypes.c_int32), ("send_to", ctypes.c_int32), ("recv_from", ctypes.c_int32)]


Step = collections.namedtuple("Step", "t kind q_chunk kv_chunk send_to recv_from")

EXPORTS = ("dfa_chunk_fwd", "dfa_chunk_fwd_acc", "dfa_chunk_fwd_batch", "dfa_span_fwd", "dfa_span_fwd_workspace",
           "dfa_chunk_fwd_form", "dfa_span_fwd_form", "dfa_chunk_bwd_form", "dfa_span_bwd_form", "dfa_merge", "dfa_merge_batch", "dfa_delta",
           "dfa_chunk_bwd",
           "dfa_chunk_bwd_batch", "dfa_chunk_bwd_workspace", "dfa_span_bwd", "dfa_span_bwd_workspace", "dfa_schedule", "dfa_schedule_mode", "dfa_schedule_window", "dfa_mfma_probe", "dfa_mfma_probe_data", "dfa_status_str",
           "dfa_version")


def lib_path() -> str:
    return _LIB_PATH


def load_library():
    """Loads libdfa.so; raises if it has not been built (no fallback path exists)."""
    global _lib
    if _lib is not None:
        return _lib
    if not os.path.exists(_LIB_PATH):
        raise RuntimeError(
            f"{_LIB_PATH} is missing: build the HIP extension first "
            "(python -c 'import __graft_entry__ as g; g.build()')")
    lib = ctypes.CDLL(_LIB_PATH)
    vp, i32, i64 = ctypes.c_void_p, ctypes.c_int32, ctypes.c_int64
    shp = ctypes.POINTER(DfaShape)
    lib.dfa_chunk_fwd.argtypes = [shp, vp, vp, vp, vp, vp, vp]
    lib.dfa_chunk_fwd_acc.argtypes = [shp, vp, vp, vp, vp, vp, vp]
    lib.dfa_merge.argtypes = [ctypes.POINTER(DfaMergeDesc), vp, vp, vp, vp, vp]
    lib.dfa_delta.argtypes = [shp, vp, vp, vp, vp]
    lib.dfa_chunk_bwd.argtypes = [shp, vp, vp, vp, vp, vp, vp, vp, vp, vp, ctypes.c_int, vp]
    lib.dfa_chunk_fwd_batch.argtypes = [shp, ctypes.POINTER(DfaFwdPair), i32, vp]
    lib.dfa_span_fwd.argtypes = [shp, ctypes.POINTER(DfaFwdSpan), i32, vp, i64, vp]
    lib.dfa_span_fwd_workspace.argtypes = [shp, ctypes.POINTER(DfaFwdSpan), i32]
    lib.dfa_chunk_fwd_form.argtypes = [shp, i32, ctypes.POINTER(DfaForm)]
    lib.dfa_chunk_bwd_form.argtypes = [shp, i32, i32, i32, i64, ctypes.POINTER(DfaForm)]
    lib.dfa_span_bwd_form.argtypes = [shp, i32, i32, i64, ctypes.POINTER(DfaForm)]
    lib.dfa_span_fwd_form.argtypes = [shp, ctypes.POINTER(DfaFwdSpan), i32, i64, ctypes.POINTER(DfaForm)]
    lib.dfa_merge_batch.argtypes = [ctypes.POINTER(DfaMergeDesc), ctypes.POINTER(DfaMergePair), i32, vp]
    lib.dfa_chunk_bwd_batch.argtypes = [shp, ctypes.POINTER(DfaBwdPair), i32, vp, i64, vp]
    lib.dfa_schedule.argtypes = [i32, i32, ctypes.POINTER(DfaStep), i32]
    lib.dfa_schedule_mode.argtypes = [i32, i32, i32, ctypes.POINTER(DfaStep), i32]
    lib.dfa_schedule_window.argtypes = [i32, i32, i32, ctypes.POINTER(DfaStep), i32]
    lib.dfa_mfma_probe.argtypes = [ctypes.c_void_p, ctypes.c_int64, i32, ctypes.POINTER(ctypes.c_double),
                                   ctypes.c_void_p]
    lib.dfa_mfma_probe_data.argtypes = [ctypes.c_void_p, ctypes.c_int64, ctypes.c_void_p, ctypes.c_int64, i32,
                                        ctypes.POINTER(ctypes.c_double), ctypes.c_void_p]
    lib.dfa_status_str.argtypes = [ctypes.c_int]
    lib.dfa_status_str.restype = ctypes.c_char_p
    lib.dfa_version.argtypes = []
    lib.dfa_span_bwd.argtypes = [shp, ctypes.POINTER(DfaBwdPair), vp, i64, vp]
    lib.dfa_span_bwd_workspace.argtypes = [shp, i32, i32]
    lib.dfa_chunk_bwd_workspace.argtypes = [shp, i32, i32, i32]
    for name in EXPORTS:
        if name not in ("dfa_status_str",):
            getattr(lib, name).restype = ctypes.c_int
    lib.dfa_chunk_bwd_workspace.restype = lib.dfa_span_fwd_workspace.restype = lib.dfa_span_bwd_workspace.restype = i64
    _lib = lib
    return lib


def dfa_status_str(status: int) -> str:
    return load_library().dfa_status_str(int(status)).decode()


def dfa_version() -> int:
    return load_library().dfa_version()


def _dt(t: torch.Tensor) -> int:
    if t.dtype == torch.bfloat16:
        return DFA_BF16
    if t.dtype == torch.float32:
        return DFA_F32
    raise TypeError(f"unsupported dtype {t.dtype}")


def _current_stream() -> int:
    return torch.cuda.current_stream().cuda_stream


if hasattr(torch._C, "_cuda_getCurrentRawStream"):      # the same without a Stream object for every launch
    def _current_stream() -> int:  # noqa: F811
        return torch._C._cuda_getCurrentRawStream(torch.cuda.current_device())


def _stream(stream) -> int:
    if stream is None:
        return _current_stream()
    return getattr(stream, "cuda_stream", stream)


def _hsd(t: torch.Tensor, name: str):
    strides = t.stride()
    if len(strides) != 3 or strides[2] != 1:
        raise ValueError(f"{name} must be [heads, seq, d] with unit innermost stride")
    return strides[:2]


def _make_shape(q, k, causal, scale, in_dtype, o=None, o_dtype=DFA_F32, lse=None, dq=None, dkv=None) -> DfaShape:
    h_q, s_q, d = q.shape
    h_kv, s_k = k.shape[:2]
    return DfaShape(h_q, h_kv, s_q, s_k, d, in_dtype, o_dtype, bool(causal), float(scale), 0, *_hsd(q, "q"), *_hsd(k, "k"),
                    *(_hsd(o, "o") if o is not None else (s_q * d, d)), lse.stride(0) if lse is not None else s_q,
                    *(_hsd(dq, "dq") if dq is not None else (s_q * d, d)),
                    *(_hsd(dkv, "dk") if dkv is not None else (s_k * d, d)))


def _check(rc: int, where: str):
    if rc != 0:
        raise DfaError(rc, where)


def dfa_chunk_fwd(q, k, v, causal, scale, o=None, lse=None, o_dtype=torch.float32, stream=None):
    """attn(q_p, k_r, v_r) of one chunk pair from the empty state -> (o, lse)."""
    lib = load_library()
    if v.shape != k.shape or v.stride() != k.stride():
        raise ValueError("k and v must share shape and strides")
    if o is None:
        o = torch.empty(q.shape, dtype=o_dtype, device=q.device)
    if lse is None:
        lse = torch.empty(q.shape[:2], dtype=torch.float32, device=q.device)
    if lse.stride(1) != 1:
        raise ValueError("lse must have unit innermost stride")
    sh = _make_shape(q, k, causal, scale, _dt(q), o=o, o_dtype=_dt(o), lse=lse)
    _check(lib.dfa_chunk_fwd(ctypes.byref(sh), q.data_ptr(), k.data_ptr(), v.data_ptr(),
                             o.data_ptr(), lse.data_ptr(), _stream(stream)), "dfa_chunk_fwd")
    return o, lse


def dfa_chunk_fwd_acc(q, k, v, causal, scale, o, lse, stream=None):
    """attn(q_p, k_r, v_r, o, s): continues from the state in (o, lse), updates both in place."""
    lib = load_library()
    if v.shape != k.shape or v.stride() != k.stride():
        raise ValueError("k and v must share shape and strides")
    if lse.stride(1) != 1:
        raise ValueError("lse must have unit innermost stride")
    sh = _make_shape(q, k, causal, scale, _dt(q), o=o, o_dtype=_dt(o), lse=lse)
    _check(lib.dfa_chunk_fwd_acc(ctypes.byref(sh), q.data_ptr(), k.data_ptr(), v.data_ptr(),
                                 o.data_ptr(), lse.data_ptr(), _stream(stream)), "dfa_chunk_fwd_acc")
    return o, lse


def dfa_merge(o_a, lse_a, o_b, lse_b, stream=None):
    """In place: (o_a, lse_a) <- merge((o_a, lse_a), (o_b, lse_b)).  Tensors [heads, seq, d] / [heads, seq]."""
    lib = load_library()
    if o_a.shape != o_b.shape or lse_a.shape != lse_b.shape or o_a.dtype != o_b.dtype:
        raise ValueError("merge operands must match")
    md = DfaMergeDesc(*o_a.shape, _dt(o_a), *_hsd(o_a, "o_a"), lse_a.stride(0), *_hsd(o_b, "o_b"), lse_b.stride(0))
    if lse_a.stride(1) != 1 or lse_b.stride(1) != 1:
        raise ValueError("lse must have unit innermost stride")
    _check(lib.dfa_merge(ctypes.byref(md), o_a.data_ptr(), lse_a.data_ptr(), o_b.data_ptr(), lse_b.data_ptr(),
                         _stream(stream)), "dfa_merge")


def dfa_delta(o, dO, delta=None, stream=None):
    """D = rowsum(dO * O) from the final merged output."""
    lib = load_library()
    if delta is None:
        delta = torch.empty(o.shape[:2], dtype=torch.float32, device=o.device)
    sh = _make_shape(dO, dO, 0, 1.0, _dt(dO), o=o, o_dtype=_dt(o), lse=delta)
    _check(lib.dfa_delta(ctypes.byref(sh), o.data_ptr(), dO.data_ptr(), delta.data_ptr(), _stream(stream)),
           "dfa_delta")
    return delta


def _same_strides(a, b) -> bool:
    """Whether the elements of a and b lie the same way (the stride of an axis of one element says nothing)."""
    x, y = a.stride(), b.stride()
    return x == y or all(n == 1 or i == j for n, i, j in zip(a.shape, x, y))


def _alike(a, b) -> bool:
    return a.shape == b.shape and _same_strides(a, b)


def _bwd_shape(q, k, v, lse, delta, dO, dq, dk, dv, causal, scale):
    """Checks that operands which share a description are alike, and describes them.  (Which outputs may be left out
    is the library's check.)"""
    if not _alike(v, k):
        raise ValueError("k and v must share shape and strides")
    if not _alike(dO, q):
        raise ValueError("dO and q must share shape and strides")
    if dk is not None and dv is not None and not _alike(dv, dk):
        raise ValueError("dk and dv must share shape and strides")
    if not _same_strides(lse, delta):
        raise ValueError("lse and delta must share strides")
    for t in (dq, dk, dv, lse, delta):
        if t is not None and t.dtype != torch.float32:
            raise TypeError("dq, dk, dv, lse, delta are fp32")
    return _make_shape(q, k, causal, scale, _dt(q), lse=lse, dq=dq, dkv=dk)


def _ptr(t):
    return None if t is None else t.data_ptr()


def _scratch(n):
    """n bytes of device memory, or None where there are not as many: scratch makes a call faster, no call needs it."""
    try:
        return torch.empty(n, dtype=torch.uint8, device="cuda")
    except torch.OutOfMemoryError:
        return None


def _workspace(n, stream):
    """Scratch of n bytes for one call on `stream`: (tensor or None, bytes).  It comes from the caching
    allocator of that stream, so that the stream's order protects it when it is let go after the call; a
    stream known by its handle alone gets none, unless it is the current one."""
    ws = None
    if n > 0 and (stream is None or _stream(stream) == _current_stream()):
        ws = _scratch(n)
    elif n > 0 and isinstance(stream, torch.cuda.Stream):
        with torch.cuda.stream(stream):
            ws = _scratch(n)
    return ws, 0 if ws is None else n


def dfa_chunk_bwd(q, k, v, lse, delta, dO, dq, dk, dv, causal, scale, accumulate=False, stream=None,
                  accumulate_dkv=None):
    """dq, dk, dv contributions of one chunk pair from the saved logsumexp and D (no forward re-run).
    dq=None computes only dk, dv; dk=dv=None computes only dq.
    accumulate_dkv: whether dk, dv are added to, where that differs from dq (None: as accumulate)."""
    lib = load_library()
    sh = _bwd_shape(q, k, v, lse, delta, dO, dq, dk, dv, causal, scale)
    pair = DfaBwdPair(q.data_ptr(), k.data_ptr(), v.data_ptr(), lse.data_ptr(), delta.data_ptr(), dO.data_ptr(),
                      _ptr(dq), _ptr(dk), _ptr(dv), bool(accumulate),
                      bool(accumulate if accumulate_dkv is None else accumulate_dkv))
    ws, n = _workspace(lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, dq is not None, dk is not None), stream)
    _check(lib.dfa_chunk_bwd_batch(ctypes.byref(sh), ctypes.byref(pair), 1, _ptr(ws), n, _stream(stream)), "dfa_chunk_bwd")
    return dq, dk, dv


def forward_form(h_q, h_kv, rows, d, dtype, causal, n_pairs):
    """The kernel form (DfaForm) of n_pairs pairs of chunks of `rows` positions as one list."""
    form, sh = DfaForm(), DfaShape(h_q, h_kv, rows, rows, d, dtype, DFA_F32, bool(causal), 1.0)
    _check(load_library().dfa_chunk_fwd_form(ctypes.byref(sh), n_pairs, ctypes.byref(form)), "dfa_chunk_fwd_form")
    return form


def sequence_form(h_q, h_kv, n, d, dtype):
    """That of a sequence of n positions as one causal call (ForwardChunks.launch, causal None)."""
    form, span = DfaForm(), DfaFwdSpan(n_keys=n, own=1)
    sh = DfaShape(h_q, h_kv, n, n, d, dtype, DFA_F32, 0, 1.0, 0, n * d, d, n * d, d)
    _check(load_library().dfa_span_fwd_form(ctypes.byref(sh), ctypes.byref(span), 1, 0, ctypes.byref(form)), "dfa_span_fwd_form")
    return form


class _Chunks:
    """Addresses of the chunks (`rows` sequence positions each) of a [heads, seq, ...] tensor.  Chunks without rows (a
    sequence shorter than its number of chunks) have none, as the empty slices of a tensor."""

    __slots__ = ("base", "step", "n")

    def __init__(self, t, rows):
        if rows < 1:
            raise DfaError(DFA_ERR_NULL, f"chunks of {rows} rows")
        self.base, self.step = t.data_ptr(), rows * t.stride(1) * t.element_size()
        self.n = t.shape[1] // rows

    def of(self, t):
        """Those of a tensor of the same shape and strides."""
        other = _Chunks.__new__(_Chunks)
        other.base, other.step, other.n = t.data_ptr(), self.step, self.n
        return other

    def __getitem__(self, i):
        if not 0 <= i < self.n:
            raise IndexError(f"chunk {i} of {self.n}")
        return self.base + i * self.step


class ForwardChunks:
    """Forward calls (dfa_chunk_fwd_batch) on the chunk pairs of whole sequences q, k, v, divided in chunks of `rows`.
    The operands are checked and described once; a launch then costs the host little more than its pointers.  An
    object serves one thread at a time."""

    def __init__(self, q, k, v, rows, scale):
        if v.shape != k.shape or v.stride() != k.stride():
            raise ValueError("k and v must share shape and strides")
        self.tensors = (q, k, v)                     # kept: launches use their addresses
        self.rows, self.lib = rows, load_library()
        self.sh = _make_shape(q, k, False, scale, _dt(q))
        self.sh.s_q = self.sh.s_k = rows
        self.q, self.k = _Chunks(q, rows), _Chunks(k, rows)
        self.v = self.k.of(v)

    def dest(self, o, lse):
        """[heads, seq, d] and [heads, seq] tensors that results can go to, in chunks of the same length."""
        if lse.stride(1) != 1:
            raise ValueError("lse must have unit innermost stride")
        return _Chunks(o, self.rows), _Chunks(lse, self.rows), (*_hsd(o, "o"), lse.stride(0)), _dt(o), (o, lse)

    def launch(self, pairs, causal, stream=None):
        """The pairs as one launch: (q_chunk, kv_chunk, dest, chunk, accumulate), the result goes to chunk number
        `chunk` of dest; accumulate: continues from the state there.  No output may overlap another pair's.
        causal None: a chunk's pair with itself is causal, no other is; pairs next to each other in the list with one
        destination, each after the first accumulating, are one walk over their key/value chunks, which
        have to be consecutive (dfa_span_fwd); one causal pair alone is a sequence that stands for the pairs of several chunks."""
        if not pairs:
            return
        sh = self.sh
        if causal is None:
            return self._launch_spans(pairs, stream)
        sh.causal, sh.o_dtype = int(bool(causal)), pairs[0][2][3]
        arr = (DfaFwdPair * len(pairs))()          # (member by member: from tuples it takes twice as long)
        for a, (qc, kc, dest, c, acc) in zip(arr, pairs):
            if dest[3] != sh.o_dtype:
                raise ValueError("outputs of a launch share their dtype")
            a.q, a.k, a.v, a.o, a.lse = self.q[qc], self.k[kc], self.v[kc], dest[0][c], dest[1][c]
            a.o_stride_h, a.o_stride_s, a.lse_stride_h = dest[2]
            a.accumulate = bool(acc)
        _check(self.lib.dfa_chunk_fwd_batch(ctypes.byref(sh), arr, len(pairs), _stream(stream)), "dfa_chunk_fwd_batch")

    def _launch_spans(self, pairs, stream):
        sh = self.sh
        sh.o_dtype = pairs[0][2][3]
        runs, kv = [], None                          # (q_chunk, dest, chunk, accumulate, key/value chunks)
        for qc, kc, dest, c, acc in pairs:
            if dest[3] != sh.o_dtype:
                raise ValueError("outputs of a launch share their dtype")
            if acc and kv is not None and (qc, c) == at and runs[-1][1] is dest:
                kv.append(kc)
            else:
                kv, at = [kc], (qc, c)
                runs.append((qc, dest, c, acc, kv))
        spans = []
        for qc, dest, c, acc, kv in runs:
            lo, hi = min(kv), max(kv)
            if hi - lo + 1 != len(kv) or len(set(kv)) != len(kv) or (qc in kv and qc != hi):
                raise ValueError("the key/value chunks of a walk are consecutive, the query chunk's own the last")
            self.k[hi]                               # (in range)
            spans.append((self.q[qc], self.k[lo], self.v[lo], dest[0][c], dest[1][c], *dest[2],
                          len(kv) * self.rows, qc == hi, bool(acc)))
        arr = (DfaFwdSpan * len(spans))(*spans)
        ws, n = _workspace(self.lib.dfa_span_fwd_workspace(ctypes.byref(sh), arr, len(spans)), stream)
        _check(self.lib.dfa_span_fwd(ctypes.byref(sh), arr, len(spans), _ptr(ws), n, _stream(stream)), "dfa_span_fwd")


def dfa_merge_batch(o, lse, rows, parts, stream=None):
    """In place: chunk c of (o, lse) <- merge(chunk c, (o_b, lse_b)) for every (c, o_b, lse_b) of parts, as one
    launch; the partials share their strides.  Partials of one chunk are next to each other in the list."""
    if not parts:
        return
    lib = load_library()
    shape, lse_shape = (o.shape[0], rows, o.shape[2]), (o.shape[0], rows)
    like, lse_like = parts[0][1].stride(), parts[0][2].stride()
    md = DfaMergeDesc(*shape, _dt(o), *_hsd(o, "o"), lse.stride(0), *_hsd(parts[0][1], "o_b"), lse_like[0])
    co, cl = _Chunks(o, rows), _Chunks(lse, rows)
    arr = (DfaMergePair * len(parts))()
    for a, (c, ob, lb) in zip(arr, parts):
        if ob.shape != shape or ob.dtype != o.dtype or ob.stride() != like or lb.shape != lse_shape or lb.stride() != lse_like:
            raise ValueError("merge operands must match")
        a.o_a, a.lse_a, a.o_b, a.lse_b = co[c], cl[c], ob.data_ptr(), lb.data_ptr()
    if lse.stride(1) != 1 or lse_like[1] != 1:
        raise ValueError("lse must have unit innermost stride")
    _check(lib.dfa_merge_batch(ctypes.byref(md), arr, len(parts), _stream(stream)), "dfa_merge_batch")


class BackwardChunks:
    """Backward calls (dfa_chunk_bwd_batch) on the chunk pairs of whole sequences, divided in chunks of `rows`; as
    ForwardChunks."""

    def __init__(self, q, k, v, lse, delta, dO, dq, dk, dv, rows, scale):
        self.tensors = (q, k, v, lse, delta, dO, dq, dk, dv)
        self.lib = load_library()
        self.sh = _bwd_shape(q, k, v, lse, delta, dO, dq, dk, dv, False, scale)
        self.sh.s_q = self.sh.s_k = rows
        by_q, by_k, by_dk = _Chunks(q, rows), _Chunks(k, rows), _Chunks(dk, rows)
        self.by_q = [by_q, _Chunks(lse, rows), _Chunks(delta, rows), by_q.of(dO), _Chunks(dq, rows)]
        self.by_kv = [by_k, by_k.of(v), by_dk, by_dk.of(dv)]

    def _pairs(self, pairs):
        arr = (DfaBwdPair * len(pairs))()
        for a, (qc, kc, acc_q, acc_kv) in zip(arr, pairs):
            a.q, a.lse, a.delta, a.dO, a.dq = (t[qc] for t in self.by_q)
            a.k, a.v, a.dk, a.dv = (t[kc] for t in self.by_kv)
            a.accumulate_dq, a.accumulate_dkv = bool(acc_q), bool(acc_kv)
        return arr

    def launch(self, pairs, causal, stream=None):
        """The pairs as one launch: (q_chunk, kv_chunk, accumulate_dq, accumulate_dkv); no query chunk and no
        key/value chunk occurs twice.  causal None: one chunk with itself, a sequence that stands for the pairs of several
        chunks (dfa_span_bwd)."""
        if not pairs:
            return
        sh = self.sh
        if causal is None:
            (qc, kc, acc_q, acc_kv), = pairs
            return self.launch_span(qc, kc, qc, acc_q, acc_kv, stream)
        sh.causal = int(bool(causal))
        arr = self._pairs(pairs)
        ws, n = _workspace(self.lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), len(pairs), 1, 1), stream)
        _check(self.lib.dfa_chunk_bwd_batch(ctypes.byref(sh), arr, len(pairs), _ptr(ws), n, _stream(stream)),
               "dfa_chunk_bwd_batch")

    def launch_span(self, qc, lo, hi, acc_q, acc_kv, stream=None):
        """Query chunk qc against the key/value chunks lo .. hi, the last of which may be its own (dfa_span_bwd)."""
        sh, rows = self.sh, self.sh.s_q
        sh.s_k, sh.causal = (hi - lo + 1) * rows, int(qc == hi)
        try:
            a = self._pairs([(qc, lo, acc_q, acc_kv)])
            self.by_kv[0][hi]                        # (in range)
            ws, n = _workspace(self.lib.dfa_span_bwd_workspace(ctypes.byref(sh), 1, 1), stream)
            _check(self.lib.dfa_span_bwd(ctypes.byref(sh), a, _ptr(ws), n, _stream(stream)), "dfa_span_bwd")
        finally:
            sh.s_k = rows


def dfa_mfma_probe(out, iters: int, stream=None) -> float:
    """Launches the register-resident MFMA stream (measurement aid); returns its FLOP count."""
    lib = load_library()
    flop = ctypes.c_double(0.0)
    _check(lib.dfa_mfma_probe(out.data_ptr(), out.numel(), int(iters), ctypes.byref(flop), _stream(stream)),
           "dfa_mfma_probe")
    return flop.value


def dfa_mfma_probe_data(operands, out, iters: int, stream=None) -> float:
    """The MFMA stream fed with the values of `operands` (a contiguous bf16 device tensor of at least
    1 MiB); returns its FLOP count."""
    lib = load_library()
    if operands.dtype != torch.bfloat16 or not operands.is_contiguous():
        raise TypeError("operands must be a contiguous bf16 tensor")
    flop = ctypes.c_double(0.0)
    _check(lib.dfa_mfma_probe_data(operands.data_ptr(), operands.numel() * 2, out.data_ptr(), out.numel(),
                                   int(iters), ctypes.byref(flop), _stream(stream)), "dfa_mfma_probe_data")
    return flop.value


def dfa_schedule(P: int, worker_id: int, mode="balanced"):
    """Step list of one worker (host integers only).  mode: "balanced", "ring", or
    ("window", window_chunks) for the local sliding window (dfa_schedule_window)."""
    # (the schedules of up to 64 workers are kept: a pass of all workers asks for each of them twice, 3 to 4 us each time)
    mode = plain_mode(mode)
    return list((_kept_steps if type(P) is int and P <= 64 else _steps)(P, worker_id, mode))


def plain_mode(mode):
    """A mode as strings and integers, which stay what they are (a window may come as a tensor or an array)."""
    if isinstance(mode, tuple):
        if mode[0] != "window":
            raise ValueError(mode)
        return "window", int(mode[1])
    return mode


def _steps(P, worker_id, mode):
    lib = load_library()
    cap = max(1, P + 1)
    buf = (DfaStep * cap)()
    if isinstance(mode, tuple):
        n = lib.dfa_schedule_window(P, worker_id, mode[1], buf, cap)
    else:
        n = lib.dfa_schedule_mode({"balanced": 0, "ring": 1}[mode], P, worker_id, buf, cap)
    if n < 0:
        raise DfaError(n, "dfa_schedule")
    return [Step(b.t, b.kind, b.q_chunk, b.kv_chunk, b.send_to, b.recv_from) for b in buf[:n]]


_kept_steps = functools.lru_cache(maxsize=256, typed=True)(_steps)
