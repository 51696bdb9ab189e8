"""Host side of the driver and the binding, without a GPU: which calls are made, and what is refused before any launch."""
import ctypes

import pytest
import torch

import paper_2310_03294_amd as dfa
from paper_2310_03294_amd import autograd, binding as B, driver

MAX_SLICE = (1 << 29) - 1       # rows * row stride (elements) of one head's slice that a call takes


def _meta(heads, n, d, pitch, dtype=torch.bfloat16):
    """A [heads, n, d] tensor with `pitch` elements between its rows, without memory."""
    return torch.empty_strided((heads, n, d), (d if pitch > d else n * d, pitch, 1), dtype=dtype, device="meta")


@pytest.fixture
def no_launches(monkeypatch):
    """The driver's calls without their launches."""
    monkeypatch.setattr(B.ForwardChunks, "launch", lambda *a, **k: None)
    monkeypatch.setattr(B.BackwardChunks, "launch", lambda *a, **k: None)
    monkeypatch.setattr(B, "dfa_merge_batch", lambda *a, **k: None)


@pytest.mark.parametrize("n,P,pitch,calls", [
    (131071, 1, 4096, 1),            # 32 heads x 128, position-major: the longest slice one call takes
    (131072, 8, 4096, 2),            # one row more than that
    (524288, 8, 4096, 8),            # every chunk needs a call of its own
    (1024, 5, 128, 1),               # 1020 rows in chunks, four left over
])
def test_delta_calls_stay_within_a_slice(monkeypatch, no_launches, n, P, pitch, calls):
    """D of a sequence longer than one call takes goes out in pieces that each stay within the limit."""
    h, c, d, seen = 2, n // P, 128, []

    def record(o, dO, delta):
        assert o.shape == dO.shape and o.shape[:2] == delta.shape
        for t in (o, dO):
            assert t.shape[1] * t.stride(1) <= MAX_SLICE
        assert o.storage_offset() // d == delta.storage_offset() == dO.storage_offset() // pitch
        seen.append((delta.storage_offset(), o.shape[1]))

    monkeypatch.setattr(B, "dfa_delta", record)
    q, k, v, dO = (_meta(h, n, d, pitch) for _ in range(4))
    driver.run_all_workers(q, k, v, dO, d ** -0.5, P, driver.Buffers(h, h, n, d, P, "meta"))
    assert len(seen) == calls and seen[0][0] == 0 and sum(rows for _, rows in seen) == c * P
    assert all(a[0] + a[1] == b[0] for a, b in zip(seen, seen[1:]))


def test_slice_limit_is_the_librarys():
    """One row more than MAX_SLICE allows is refused (before any launch)."""
    rows, pitch = 131072, 4096
    assert rows * pitch == MAX_SLICE + 1
    sh = B.DfaShape(h_q=1, h_kv=1, s_q=rows, s_k=rows, d=128, dtype=B.DFA_BF16, o_dtype=B.DFA_F32, scale=1.0, q_stride_h=128,
                    q_stride_s=pitch, kv_stride_h=128, kv_stride_s=pitch, o_stride_h=rows * 128, o_stride_s=128,
                    lse_stride_h=rows)
    assert dfa.load_library().dfa_delta(ctypes.byref(sh), 4096, 4096, 4096, None) == -2


@pytest.mark.parametrize("mode", ["balanced", "ring"])
def test_sequence_shorter_than_its_chunks_is_refused(mode):
    """Chunks without rows: no pass may return as if it had written its outputs."""
    n, P, h, d = 3, 4, 2, 64
    q, k, v, do = (torch.zeros(h, n, d) for _ in range(4))
    bufs = driver.Buffers(h, h, n, d, P, "cpu")
    calls = [lambda: driver.run_all_workers(q, k, v, do, 1.0, P, bufs, mode, backward=False),
             lambda: driver.forward_worker(q, k, v, 1.0, P, P - 1, bufs, mode=mode),
             lambda: driver.backward_all_workers(q, k, v, do, 1.0, P, bufs, mode),
             lambda: driver.backward_worker(q, k, v, do, 1.0, P, P - 1, bufs, mode),
             lambda: autograd.dist_flash_attn(q, k, v, 1.0, P)]
    for call in calls:
        with pytest.raises(dfa.DfaError) as e:
            call()
        assert e.value.status == -1


def _bwd_operands(h, n, d=64):
    """q, k, v, lse, delta, dO, dq, dk, dv, all contiguous."""
    x = {t: torch.zeros(h, n, d) for t in ("q", "k", "v", "dO", "dq", "dk", "dv")}
    return {**x, "lse": torch.zeros(h, n), "delta": torch.zeros(h, n)}


def _shape_of(x):
    return B._bwd_shape(*(x[t] for t in ("q", "k", "v", "lse", "delta", "dO", "dq", "dk", "dv")), False, 1.0)


@pytest.mark.parametrize("name", ["dO", "v", "dv", "delta"])
def test_strides_of_one_head_do_not_matter(name):
    """With one head the head stride is never used: slices of larger tensors next to contiguous ones.  With two it is,
    and operands that share a description have to share it."""
    for h in (1, 2):
        x = _bwd_operands(h, 8)
        x[name] = torch.zeros(h, 16, *x[name].shape[2:])[:, :8]
        if h == 1:
            assert _shape_of(x).h_q == 1
            B.BackwardChunks(*(x[t] for t in ("q", "k", "v", "lse", "delta", "dO", "dq", "dk", "dv")), 4, 1.0)
        else:
            with pytest.raises(ValueError):
                _shape_of(x)
    x = _bwd_operands(1, 8)
    x["q"] = torch.zeros(8, 1, 64).transpose(0, 1)        # position-major: contiguous all the same
    assert x["q"].is_contiguous() and x["q"].stride() != x["dO"].stride()
    assert _shape_of(x).s_q == 8


@pytest.mark.parametrize("missing", [("dq", "dk", "dv"), ("dk",), ("dv",), ("dq", "dv")])
def test_missing_outputs_are_refused_by_the_library(missing):
    x = _bwd_operands(2, 8)
    for t in missing:
        x[t] = None
    with pytest.raises(dfa.DfaError) as e:
        dfa.dfa_chunk_bwd(*(x[t] for t in ("q", "k", "v", "lse", "delta", "dO", "dq", "dk", "dv")), False, 1.0, stream=0)
    assert e.value.status == -1


@pytest.mark.parametrize("mode,P", [("ring", 4), (("window", 2), 4), ("balanced", 2)])
def test_buffers_of_the_caller_without_partials(monkeypatch, no_launches, mode, P):
    """A schedule without helpers needs no partial buffers: O and L of the caller's own are enough."""
    monkeypatch.setattr(B, "dfa_delta", lambda *a, **k: None)
    h, n, d = 2, 64, 64
    q, k, v, do = (torch.zeros(h, n, d) for _ in range(4))
    bufs = driver.Buffers(h, h, n, d, P, "cpu", outputs=False)
    bufs.O, bufs.L = torch.zeros(h, n, d), torch.zeros(h, n)
    driver.run_all_workers(q, k, v, do, 1.0, P, bufs, mode)


def test_backward_without_memory_for_scratch(monkeypatch):
    """Scratch that cannot be had is done without."""
    def empty(*a, **k):
        raise torch.OutOfMemoryError

    monkeypatch.setattr(B, "_current_stream", lambda: 0)
    monkeypatch.setattr(torch, "empty", empty)
    assert B._workspace(1 << 20, None) == B._workspace(1 << 20, 0) == (None, 0)


@pytest.mark.parametrize("extra", [0, 1, 100])
@pytest.mark.parametrize("P", [3, 8, 11])
def test_fewer_partials_than_helpers(monkeypatch, P, extra):
    """Memory for `extra` more partial buffers than the first: every pair is still computed once, and no buffer is
    written again before it is merged."""
    h, c, d = 2, 4, 64
    bufs = driver.Buffers(h, h, P * c, d, P, "cpu", grads=False)
    like, left = torch.empty_like, [2 * extra]

    def empty_like(t):
        left[0] -= 1
        if left[0] < 0:
            raise torch.OutOfMemoryError
        return like(t)

    pairs, waiting = [], set()

    def launch(self, items, causal, stream=None):
        for q, kv, dest, _, _ in items:
            pairs.append((q, kv))
            if dest[4][0] is not bufs.O:
                assert id(dest[4][0]) not in waiting
                waiting.add(id(dest[4][0]))

    def merge(o, lse, rows, parts, stream=None):
        assert {id(ob) for _, ob, _ in parts} == waiting and len(waiting) == len(parts)
        waiting.clear()

    monkeypatch.setattr(torch, "empty_like", empty_like)
    monkeypatch.setattr(B.ForwardChunks, "launch", launch)
    monkeypatch.setattr(B, "dfa_merge_batch", merge)
    q, k, v = (torch.zeros(h, P * c, d) for _ in range(3))
    driver.run_all_workers(q, k, v, None, 1.0, P, bufs, backward=False)
    assert sorted(pairs) == [(i, j) for i in range(P) for j in range(i + 1)] and not waiting
    assert len(bufs.part_o) == len(bufs.part_l) == min(1 + extra, max(1, (P - 1) // 2))
