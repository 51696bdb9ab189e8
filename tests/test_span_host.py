"""Host side of walks over several key/value chunks, without a GPU: which pairs the driver computes, and what is refused."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2310_03294_amd as dfa
import test_gpu_spans
from paper_2310_03294_amd import binding as B, driver


def _tensors(h, n, d=64):
    return [torch.zeros(h, n, d) for _ in range(4)]


@pytest.mark.parametrize("P", [1, 2, 3, 4, 7, 8, 16])
def test_share_computes_the_schedules_pairs(monkeypatch, P):
    """Forward and backward of a share: every pair of the worker's schedule once, every partial merged, D before the backward."""
    h, c, d = 2, 4, 64
    q, k, v, do = _tensors(h, P * c)
    log = []

    def span(self, qc, lo, hi, acc_q, acc_kv, stream=None):
        assert not acc_q and not acc_kv and lo < hi
        log.extend(("bwd", qc, kc) for kc in range(lo, hi + 1))

    def pairs(self, items, causal, stream=None):
        if causal:      # its own chunk alone: a pair, not a sequence of several chunks
            assert items == [(w, w, False, False)]
        assert causal or all(acc_kv and not acc_q for _, _, acc_q, acc_kv in items)
        log.extend(("bwd", qc, kc) for qc, kc, _, _ in items)

    monkeypatch.setattr(B.ForwardChunks, "launch", lambda self, items, causal, stream=None: log.extend(
        ("fwd", qc, kc, dest[4][0] is bufs.O, acc) for qc, kc, dest, _, acc in items if causal is (None if len(items) > 1 else True)))
    monkeypatch.setattr(B.BackwardChunks, "launch_span", span)
    monkeypatch.setattr(B.BackwardChunks, "launch", pairs)
    monkeypatch.setattr(B, "dfa_merge_batch", lambda o, lse, rows, parts: log.extend(("merge", i) for i, _, _ in parts))
    monkeypatch.setattr(B, "dfa_delta", lambda *a, **kw: log.append("delta"))
    for w in range(P):
        bufs = driver.Buffers(h, h, P * c, d, P, "cpu")
        sched = dfa.dfa_schedule(P, w)
        remote = {st.recv_from: (bufs.part_o[0], bufs.part_l[0]) for st in sched if st.recv_from >= 0}
        log.clear()
        driver.run_worker_share(q, k, v, do, 1.0, P, w, bufs, remote)
        mine = sorted((st.q_chunk, st.kv_chunk) for st in sched if st.kind != B.DFA_STEP_IDLE)
        fwd = [x for x in log if x[0] == "fwd"]
        assert sorted(x[1:3] for x in fwd) == mine and sorted(x[1:] for x in log if x[0] == "bwd") == mine
        assert all(x[3] == (x[1] == w) and x[4] == (x[1] == w != x[2]) for x in fwd)
        assert log.count(("merge", w)) == len(remote) and log.count("delta") == 1
        assert log.index("delta") == len(fwd) + len(remote)


@pytest.mark.parametrize("h_q,h_kv,c,span", [(16, 4, 6000, False), (8, 2, 8192, False), (4, 4, 16384, False), (16, 4, 4096, True), (32, 8, 8192, True),
                                             (2, 1, 8192, True)])
def test_backward_of_long_chunks_of_few_heads_goes_pair_by_pair(monkeypatch, h_q, h_kv, c, span):
    """(Its walk leaves the XCDs unequal shares, and the pairs fill the device.)  Every pair once, dq of the first overwritten."""
    P, log = 4, []
    q, k = (torch.empty(h, P * c, 128, dtype=torch.bfloat16, device="meta") for h in (h_q, h_kv))
    bufs = driver.Buffers(h_q, h_kv, P * c, 128, P, "meta")
    monkeypatch.setattr(B, "dfa_delta", lambda *a, **kw: None)
    monkeypatch.setattr(B.BackwardChunks, "launch_span", lambda self, qc, lo, hi, acc_q, acc_kv, stream=None: log.append("span"))
    monkeypatch.setattr(B.BackwardChunks, "launch", lambda self, items, causal, stream=None: log.extend((*x, causal) for x in items))
    driver._backward_at_hand(q, k, k, q, 1.0, dfa.dfa_schedule(P, P - 1), P - 1, bufs)
    assert log == (["span"] if span else [(3, 3, False, False, True), (3, 2, True, False, False), (3, 1, True, False, False)])


def test_divisions_of_the_backward():
    """What a pair of chunks asks for in scratch: as before there were spans where sharing dq's walk gains little (its 128-row form
    has no scratch), its sums where it gains much; spans divide more."""
    lib = dfa.load_library()

    def ask(h_q, h_kv, s_q, s_k, span):
        sh = B.DfaShape(h_q=h_q, h_kv=h_kv, s_q=s_q, s_k=s_k, d=128, dtype=B.DFA_BF16, scale=1.0, causal=span)
        if span:
            return lib.dfa_span_bwd_workspace(ctypes.byref(sh), 1, 1)
        return lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, 1, 1)

    for shape in ((8, 8, 1000, 2500), (16, 4, 1024, 4096), (16, 4, 2048, 8192), (8, 2, 4096, 16384), (32, 8, 1024, 4096)):
        assert ask(*shape, 0) == 0, shape
    for shape in ((1, 1, 1000, 30000), (8, 8, 128, 8000), (32, 32, 128, 20000)):
        assert ask(*shape, 0) > 0, shape
    for shape in ((4, 1, 8192, 40960), (8, 2, 4096, 20480), (8, 2, 700, 3500)):
        assert ask(*shape, 1) > 0, shape


def test_divisions_of_short_backward_calls():
    """(rows of dq's workgroups, workgroups per key tile) where the wrong ones cost 10 % and more.  us, with one, two or four per tile as
    an estimate by even shares chose / so: 32 over 8 heads x 640 diagonal 39.2 / 32.9, one head x 3000 72.8 / 61.6, 16 over 4 x 2304 182.6
    / 142.7, x 1500 diagonal 65.7 / 57.2, 32 over 8 x 1280 118.6 / 102.0; and calls that are right undivided."""
    lib, form = dfa.load_library(), B.DfaForm()
    for shape, want in (((32, 8, 640, 640, 1), (128, 3)), ((1, 1, 3000, 3000, 0), (128, 2)), ((1, 1, 1500, 1500, 1), (128, 2)),
                        ((16, 4, 2304, 2304, 0), (128, 3)), ((16, 4, 1500, 1500, 1), (128, 3)), ((32, 8, 1280, 1280, 0), (256, 4)),
                        ((8, 8, 1000, 1900, 0), (128, 1)), ((32, 32, 1024, 1024, 1), (128, 1)), ((32, 32, 4096, 4096, 0), (256, 1))):
        h_q, h_kv, s_q, s_k, causal = shape
        sh = B.DfaShape(h_q=h_q, h_kv=h_kv, s_q=s_q, s_k=s_k, d=128, dtype=B.DFA_BF16, scale=1.0, causal=causal)
        assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, 128 << 20, ctypes.byref(form)) == 0
        assert (form.rows, form.cuts) == want, shape
        assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, 0, ctypes.byref(form)) == 0 and form.cuts == 1


def test_divisions_of_short_walks_by_both_kinds_parts():
    """(workgroups per key tile, per row tile of dq) where the first division of dk, dv with dq's in parts is far from the best one.  us,
    in the division that a search cut off there found / so: 4 heads over 1 x 1571 rows x 4713 keys 89.0 / 61.5, 4 over 1 x 1645 x 3290
    67.5 / 55.0, 32 over 1 x 84 x 2941 58.5 / 37.3."""
    lib, form = dfa.load_library(), B.DfaForm()
    for shape, want in (((4, 1, 1571, 4713), (4, 2)), ((4, 1, 1645, 3290), (4, 2)), ((32, 1, 84, 2941), (6, 3))):
        h_q, h_kv, s_q, s_k = shape
        sh = B.DfaShape(h_q=h_q, h_kv=h_kv, s_q=s_q, s_k=s_k, d=128, dtype=B.DFA_BF16, scale=1.0)
        assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, 128 << 20, ctypes.byref(form)) == 0
        assert (form.cuts, form.q_cuts) == want, shape


def test_forms_of_dq_alone():
    """256 rows where they are the faster ones: long walks and whole rounds of the device; a list of 16 pairs of 32 heads x 128 rows takes
    1.7 times as long with them, 32 heads x 5000 rows 1.1, x 2048 keys 1.05."""
    lib, form = dfa.load_library(), B.DfaForm()
    for shape, rows in (((32, 32, 16384, 16384, 1), 256), ((32, 8, 8192, 8192, 1), 256), ((32, 32, 4096, 20480, 1), 256), ((32, 32, 2048, 8192, 1), 256),
                        ((8, 2, 10000, 16384, 4), 256), ((32, 8, 128, 128, 16), 128), ((32, 32, 1024, 1024, 4), 128), ((32, 32, 5000, 25000, 1), 128),
                        ((32, 32, 4096, 4096, 1), 128), ((16, 4, 6000, 6000, 4), 128), ((32, 32, 2100, 16384, 1), 128)):
        h_q, h_kv, s_q, s_k, n = shape
        sh = B.DfaShape(h_q=h_q, h_kv=h_kv, s_q=s_q, s_k=s_k, d=128, dtype=B.DFA_BF16, scale=1.0)
        assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), n, 1, 0, 0, ctypes.byref(form)) == 0
        assert (form.rows, form.parts, form.cuts, form.q_cuts) == (rows, 1, 1, 1), shape


def test_forms_of_the_f32_diagonal():
    """Short diagonals of few heads are in the 4-part form without scratch; with scratch the walks are shared where it gains (8 heads x 512
    60.7 us in 4 parts, 51.1 in two, both walks shared; 8 over 2 x 2048 at d = 64 182 with 6 shares, 163 with 4)."""
    lib, form = dfa.load_library(), B.DfaForm()

    def of(h_q, h_kv, s, d, ws):
        sh = B.DfaShape(h_q=h_q, h_kv=h_kv, s_q=s, s_k=s, d=d, dtype=B.DFA_F32, scale=1.0, causal=1)
        assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, ws, ctypes.byref(form)) == 0
        return form.parts, form.cuts, form.q_cuts

    for shape in ((1, 1, 256, 128), (1, 1, 1024, 128), (8, 8, 128, 128), (8, 8, 512, 128), (8, 2, 512, 128), (8, 2, 1024, 128), (32, 8, 128, 128)):
        assert of(*shape, 0) == (4, 1, 1), shape
    for shape, want in (((8, 8, 128, 128), (2, 3, 2)), ((8, 8, 512, 128), (2, 2, 2)), ((8, 2, 512, 128), (2, 8, 2)), ((32, 8, 128, 128), (4, 4, 1)),
                        ((8, 2, 512, 64), (4, 6, 1)), ((8, 2, 2048, 64), (2, 4, 1)), ((4, 4, 1024, 128), (2, 3, 2)), ((4, 4, 1536, 128), (2, 2, 2)),
                        ((32, 8, 333, 128), (1, 6, 1)), ((1, 1, 1024, 128), (4, 4, 4)), ((1, 1, 1024, 64), (4, 4, 4))):
        assert of(*shape, 128 << 20) == want, shape
    sh = B.DfaShape(h_q=8, h_kv=8, s_q=512, s_k=512, d=128, dtype=B.DFA_F32, scale=1.0, causal=1)      # a sequence: sums, no 4 parts
    assert lib.dfa_span_bwd_form(ctypes.byref(sh), 1, 1, 0, ctypes.byref(form)) == 0 and form.parts == 2
    bad = lambda n=1, dq=1, dk=1, ws=0, f=ctypes.byref(form): lib.dfa_chunk_bwd_form(ctypes.byref(sh), n, dq, dk, ws, f)
    assert bad(n=0) == bad(ws=-1) == bad(dq=0, dk=0) == -4 and bad(f=None) == -1


def test_long_sequences_stay_step_by_step(monkeypatch):
    """A walk longer than a call's slice is not one call: the time steps' lists, each way."""
    h, d, P, c = 2, 128, 4, 45000
    t = torch.empty_strided((h, P * c, d), (d, 4096, 1), dtype=torch.bfloat16, device="meta")
    assert len(dfa.dfa_schedule(P, 0)) * c * 4096 > B.MAX_SLICE >= c * 4096
    calls = []
    monkeypatch.setattr(B.ForwardChunks, "launch", lambda self, items, causal, stream=None: items and calls.append(("fwd", causal, len(items))))
    monkeypatch.setattr(B.BackwardChunks, "launch", lambda self, items, causal, stream=None: items and calls.append(("bwd", causal, len(items))))
    monkeypatch.setattr(B, "dfa_merge_batch", lambda *a, **kw: None)
    monkeypatch.setattr(B, "dfa_delta", lambda *a, **kw: None)
    bufs = driver.Buffers(h, h, P * c, d, P, "meta")
    driver.run_all_workers(t, t, t, t, 1.0, P, bufs)
    _assert_time_steps(calls, P)


def _assert_time_steps(calls, P):
    """The launches of the balanced schedule of P = 4 workers: lists of diagonal pairs, of the owners' and helpers' pairs."""
    assert P == 4
    assert [x[1:] for x in calls if x[0] == "fwd"] == [(True, 4), (False, 4), (False, 2)]
    assert [x[1:] for x in calls if x[0] == "bwd"] == [(True, 4), (False, 3), (False, 1), (False, 2)]


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
def test_the_schedule_as_it_is_written(monkeypatch, dtype):
    """at_once=False: pairs of time steps and merges of partials, fused or pair by pair; by default neither."""
    h, d, P, c, calls = 2, 128, 4, 64, []
    t = torch.empty((h, P * c, d), dtype=dtype, device="meta")
    monkeypatch.setattr(B.ForwardChunks, "launch", lambda self, items, causal, stream=None: items and calls.append(("fwd", causal, len(items))))
    monkeypatch.setattr(B.BackwardChunks, "launch", lambda self, items, causal, stream=None: items and calls.append(("bwd", causal, len(items))))
    monkeypatch.setattr(B, "dfa_merge_batch", lambda o, l, rows, parts: parts and calls.append(("merge", len(parts))))
    monkeypatch.setattr(B, "dfa_merge", lambda *a, **kw: calls.append(("merge", 1)))
    monkeypatch.setattr(B, "dfa_chunk_fwd", lambda *a, **kw: calls.append(("pair",)))
    monkeypatch.setattr(B, "dfa_delta", lambda *a, **kw: None)
    bufs = driver.Buffers(h, h, P * c, d, P, "meta")
    driver.run_all_workers(t, t, t, t, 1.0, P, bufs, at_once=False)
    _assert_time_steps(calls, P)
    assert [x for x in calls if x[0] == "merge"] == [("merge", 1)]
    calls.clear()
    driver.run_all_workers(t, t, t, t, 1.0, P, bufs, fused=False)
    assert calls.count(("pair",)) == 10 and calls.count(("merge", 1)) == 6
    assert [x[1:] for x in calls if x[0] == "bwd"] == [(True, 4), (False, 3), (False, 1), (False, 2)]
    calls.clear()
    driver.run_all_workers(t, t, t, t, 1.0, P, bufs)
    assert [x for x in calls if x[0] == "bwd"] == [("bwd", None, 1)] and len([x for x in calls if x[0] == "fwd"]) == 1


@pytest.mark.parametrize("mode", ["balanced", "ring", ("window", 1), ("window", 3)])
@pytest.mark.parametrize("P", [1, 2, 3, 4, 8, 16])
def test_no_way_of_all_workers_drops_remainders(P, mode):
    """bf16: where a list of pairs of a time step is in the 64-row form (weights of 16 bits), the one call or the walks that stand for it
    are; the time steps are what they are."""
    lib, seen = dfa.load_library(), set()
    for h_q, h_kv in ((1, 1), (2, 1), (8, 8), (16, 4), (32, 8), (48, 16), (64, 64)):
        for c in (1, 64, 65, 100, 128, 257, 300, 512, 513, 700, 1000, 1023, 2047, 2048, 2049, 4096, 9000):
            scheds = [dfa.dfa_schedule(P, w, mode) for w in range(P)]
            rows = {}
            for t, steps in enumerate(zip(*scheds)):
                n = sum(st.kind != B.DFA_STEP_IDLE for st in steps)
                rows[t] = B.forward_form(h_q, h_kv, c, 128, B.DFA_BF16, t == 0, n).rows if n else 0
            bufs = driver.Buffers(h_q, h_kv, P * c, 128, P, "meta")
            q, k = (torch.empty(h, P * c, 128, dtype=torch.bfloat16, device="meta") for h in (h_q, h_kv))
            one, walks = driver._how_at_once(q, k, bufs, P, mode)
            seen.add((one, walks))
            full = any(r == 64 for t, r in rows.items() if t)
            if one and P > 1:
                assert 64 not in rows.values() or B.sequence_form(h_q, h_kv, P * c, 128, B.DFA_BF16).rows == 64, (h_q, c)
            elif not one and walks:
                spans = [(sum(st.kind in (B.DFA_STEP_DIAG, B.DFA_STEP_OWN) for st in s) * c, 1) for s in scheds]
                spans += [(c, 0) for s in scheds for st in s if st.kind == B.DFA_STEP_HELP]
                arr = (B.DfaFwdSpan * len(spans))(*[B.DfaFwdSpan(n_keys=n, own=own) for n, own in spans])
                sh, form = B.DfaShape(h_q, h_kv, c, c, 128, B.DFA_BF16, B.DFA_F32, 0, 1.0, 0, P * c * 128, 128, P * c * 128, 128), B.DfaForm()
                assert lib.dfa_span_fwd_form(ctypes.byref(sh), arr, len(spans), 0, ctypes.byref(form)) == 0
                assert not full or form.rows == 64, (h_q, c)
    assert (True, True) in seen or isinstance(mode, tuple)


@pytest.mark.parametrize("dtype,d,h_q,h_kv,c,walks,acc,form", test_gpu_spans.FWD)
def test_walks_take_the_forms_they_are_tested_in(dtype, d, h_q, h_kv, c, walks, acc, form):
    """The table of the GPU tests, with all the scratch that is asked for: a change of the estimates shows here."""
    lib, got, n = dfa.load_library(), B.DfaForm(), max(w[0] for w in walks) + 1
    arr = (B.DfaFwdSpan * len(walks))(*[B.DfaFwdSpan(n_keys=(hi - lo + 1) * c, own=hi == qc, accumulate=i in acc)
                                        for i, (qc, lo, hi) in enumerate(walks)])
    sh = B.DfaShape(h_q, h_kv, c, c, d, B.DFA_BF16 if dtype == torch.bfloat16 else B.DFA_F32, B.DFA_F32, 0, d ** -0.5, 0, n * c * d, d,
                    n * c * d, d)
    ws = lib.dfa_span_fwd_workspace(ctypes.byref(sh), arr, len(walks))
    assert lib.dfa_span_fwd_form(ctypes.byref(sh), arr, len(walks), ws, ctypes.byref(got)) == 0
    assert (got.rows, got.parts, got.cuts) == form and (ws > 0) == (form[2] > 1)


def test_every_form_of_walks_is_tested():
    forms = {(dtype, d, form[:2]) for dtype, d, _, _, _, _, _, form in test_gpu_spans.FWD}
    bf16, f32 = torch.bfloat16, torch.float32
    assert forms == {(bf16, 128, x) for x in ((64, 4), (128, 2), (256, 1))} | {(f32, d, x) for d in (64, 128) for x in ((32, 4), (64, 2))}


@pytest.mark.parametrize("pairs", [
    [(2, 2, False), (2, 0, True)],                 # a chunk is left out
    [(1, 1, False), (1, 2, True)],                 # keys behind the query chunk's own
])
def test_walks_of_other_chunks_are_refused(pairs):
    q, k, v, _ = _tensors(2, 16)
    fwd = B.ForwardChunks(q, k, v, 4, 1.0)
    dest = fwd.dest(torch.zeros(2, 16, 64), torch.zeros(2, 16))
    with pytest.raises(ValueError):
        fwd.launch([(qc, kc, dest, qc, acc) for qc, kc, acc in pairs], None)


def test_span_arguments():
    """Refused before any launch: status codes of dfa_span_fwd and dfa_span_bwd."""
    lib = dfa.load_library()

    def shape(**kw):
        sh = B.DfaShape(h_q=2, h_kv=2, s_q=64, s_k=64, d=64, dtype=B.DFA_F32, o_dtype=B.DFA_F32, scale=1.0, q_stride_h=4096,
                        q_stride_s=64, kv_stride_h=1 << 20, kv_stride_s=64, o_stride_h=4096, o_stride_s=64, lse_stride_h=64,
                        dq_stride_h=4096, dq_stride_s=64, dkv_stride_h=1 << 20, dkv_stride_s=64)
        for a, b in kw.items():
            setattr(sh, a, b)
        return sh

    def fwd(sh=None, n=1, ws=None, ws_bytes=0, **kw):
        x = B.DfaFwdSpan(4096, 4096, 4096, 4096, 4096, 4096, 64, 64, 128, 1, 0, 0)
        for a, b in kw.items():
            setattr(x, a, b)
        return lib.dfa_span_fwd(ctypes.byref(sh or shape()), ctypes.byref(x), n, ws, ws_bytes, None)

    assert fwd(n=0) == 0 and fwd(n=-1) == -4 and fwd(sh=shape(s_q=0)) == 0
    for f in ("q", "k", "v", "o", "lse"):
        assert fwd(**{f: None}) == -1
    assert fwd(q=4100) == -2 and fwd(n_keys=0) == -2 and fwd(n_keys=1 << 24) == -2 and fwd(sh=shape(q_stride_s=63)) == -2
    assert fwd(n_keys=63) == -4 and fwd(reserved=1) == -4 and fwd(ws_bytes=-1) == -4 and fwd(ws=8, ws_bytes=64) == -2
    assert fwd(sh=shape(dtype=7)) == -3 and fwd(sh=shape(d=96)) == -2 and fwd(o_stride_s=60) == -2
    x = B.DfaFwdSpan(4096, 4096, 4096, 4096, 4096, 4096, 64, 64, 1280, 1, 0, 0)
    assert lib.dfa_span_fwd_workspace(ctypes.byref(shape()), ctypes.byref(x), 1) > 0
    assert lib.dfa_span_fwd_workspace(ctypes.byref(shape(scale=-1.0)), ctypes.byref(x), 1) == -4

    def bwd(sh, **kw):
        y = B.DfaBwdPair(*[4096] * 9, 0, 0)
        for a, b in kw.items():
            setattr(y, a, b)
        return lib.dfa_span_bwd(ctypes.byref(sh), ctypes.byref(y), None, 0, None)

    assert bwd(shape(s_k=63, causal=1)) == -4 and bwd(shape(s_k=128, causal=1), dk=None) == -1
    assert bwd(shape(s_k=128, causal=1), q=None) == -1 and bwd(shape(s_k=128, causal=2)) == -4
    assert lib.dfa_span_bwd_workspace(ctypes.byref(shape(s_k=4096, causal=1)), 1, 1) > 0
    # what a pair's backward refused it still refuses
    y = B.DfaBwdPair(*[4096] * 9, 0, 0)
    assert lib.dfa_chunk_bwd_batch(ctypes.byref(shape(s_k=128, causal=1)), ctypes.byref(y), 1, None, 0, None) == -4


def test_a_schedule_is_that_of_the_mode_as_it_is_now():
    """Kept schedules go by the window's value; a window comes as any kind of number."""
    window = torch.tensor(1)
    for n in (1, 4):
        window.fill_(n)
        assert dfa.dfa_schedule(8, 7, ("window", window)) == dfa.dfa_schedule(8, 7, ("window", np.array(n))) == dfa.dfa_schedule(8, 7, ("window", n))
        assert len(dfa.dfa_schedule(8, 7, ("window", n))) == n + 1
    for bad, error in ((("other", 1), ValueError), ("other", KeyError)):
        with pytest.raises(error):
            dfa.dfa_schedule(8, 7, bad)


def test_a_schedule_is_the_callers_own():
    want = [tuple(st) for st in dfa.dfa_schedule(8, 3)]
    dfa.dfa_schedule(8, 3).clear()
    assert [tuple(st) for st in dfa.dfa_schedule(8, 3)] == want
    for bad in ((8.0, 3), (8, 3.0), (8, 8), (0, 0), (8, -1)):      # refused, also where an equal number has been asked for
        with pytest.raises((ctypes.ArgumentError, TypeError, dfa.DfaError)):
            dfa.dfa_schedule(*bad)
