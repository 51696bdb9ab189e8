"""GPU parity of lists of pairs (one launch for the pairs of a time step) in every kernel form that a list reaches, and of
the backward with any amount of scratch; against the fp64 oracle (bounds as in the parity tests)."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2310_03294_amd as dfa
from paper_2310_03294_amd import binding as B, driver
from gpu_util import TOL, case, dev, maxerr, np64
from oracle import attention as A

pytestmark = pytest.mark.gpu

BF16, F32 = torch.bfloat16, torch.float32


def _slices(t, i, c):
    return t[:, i * c:(i + 1) * c]


def _pairs(n, causal):
    """Query chunk i with key/value chunk n - 1 - i (diagonal: i)."""
    return [(i, i if causal else n - 1 - i) for i in range(n)]


# heads, chunk, pairs, causal; the form that the number of workgroups of all pairs selects
FWD = [
    (BF16, 4, 2, 450, 4, False),      # 64 rows, 4 key parts
    (BF16, 16, 16, 450, 4, False),    # 128 rows, 2 key parts: 256 workgroups
    (BF16, 32, 16, 300, 9, False),    # 128 rows: 576 workgroups of 256 rows would leave a last round of 64
    (BF16, 32, 32, 300, 4, False),    # 256 rows, ragged
    (BF16, 32, 8, 320, 4, False),     # 256 rows, whole tiles
    (BF16, 4, 2, 450, 4, True),       # 64 rows, 4 key parts
    (BF16, 16, 4, 300, 4, True),      # 128 rows
    (BF16, 8, 2, 1100, 3, True),      # 128 rows, 2 key parts: 216 workgroups
    (BF16, 32, 32, 300, 4, True),     # 128 rows: 384 workgroups
    (BF16, 3, 1, 70, 19, True),       # more pairs than a launch takes
    (F32, 40, 20, 150, 4, False),     # 2 parts
    (F32, 130, 130, 150, 2, False),   # 1 part
    (F32, 10, 5, 150, 3, True),       # 4 parts
]


@pytest.mark.parametrize("dtype,h_q,h_kv,c,n,causal", FWD)
def test_forward_lists(dtype, h_q, h_kv, c, n, causal):
    """Every second pair continues from a state in a chunk of a whole sequence, the others go to buffers of their own."""
    d, tol = 128, TOL[dtype]
    scale = d ** -0.5
    q, k, v, _ = case(100 + c + h_q, h_q, h_kv, n * c, n * c, d, dtype)
    o0, lse0 = torch.randn(h_q, n * c, d) * 0.1, torch.randn(h_q, n * c) + 5
    O, L = o0.to(dev()), lse0.to(dev())
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    fwd = B.ForwardChunks(Q, K, V, c, scale)
    state, pairs = fwd.dest(O, L), _pairs(n, causal)
    own = {i: (torch.empty(h_q, c, d, device=dev()), torch.empty(h_q, c, device=dev())) for i in range(1, n, 2)}
    fwd.launch([(qc, kc, fwd.dest(*own[qc]), 0, False) if qc in own else (qc, kc, state, qc, True) for qc, kc in pairs],
               causal)
    for qc, kc in pairs:
        want = A.attention_fwd(np64(_slices(q, qc, c)), np64(_slices(k, kc, c)), np64(_slices(v, kc, c)), scale, causal=causal)
        if qc not in own:
            want = A.merge(np64(_slices(o0, qc, c)), np64(_slices(lse0, qc, c)), *want)
        o, lse = own[qc] if qc in own else (_slices(O, qc, c), _slices(L, qc, c))
        assert maxerr(o, want[0]) <= tol and maxerr(lse, want[1]) <= tol
    for i in own:       # the state of these chunks is not theirs to write
        assert torch.equal(_slices(O, i, c).cpu(), _slices(o0, i, c)) and torch.equal(_slices(L, i, c).cpu(), _slices(lse0, i, c))


def test_forward_list_of_long_diagonal_chunks():
    """256-row workgroups on the diagonal chunks of three pairs, by sampled rows."""
    h_q, c, n, d, tol = 8, 6144, 3, 128, TOL[BF16]
    q, k, v, _ = case(7, h_q, 1, n * c, n * c, d, BF16)
    fwd = B.ForwardChunks(*(t.to(dev()) for t in (q, k, v)), c, d ** -0.5)
    O, L = torch.empty(h_q, n * c, d, device=dev()), torch.empty(h_q, n * c, device=dev())
    fwd.launch([(i, i, fwd.dest(O, L), i, False) for i in range(n)], True)
    rows = sorted({0, 1, 63, 64, 255, 256, c // 2, c - 257, c - 65, c - 1})
    for i in range(n):
        for h in (0, h_q - 1):
            o, lse = _slices(O, i, c)[h, rows], _slices(L, i, c)[h, rows]
            want = A.rows_fwd(np64(_slices(q, i, c)[h, rows]), rows, np64(_slices(k, i, c)[0]), np64(_slices(v, i, c)[0]), d ** -0.5)
            assert maxerr(o, want[0]) <= tol and maxerr(lse, want[1]) <= 1e-4


class _Backward:
    """A list of pairs with the logsumexp and D that each pair's own keys give, and the oracle's gradients."""

    def __init__(self, dtype, h_q, h_kv, c, n, causal, d=128, seed=300, only=None):
        self.scale, self.c, self.n, self.causal = d ** -0.5, c, n, causal
        q, k, v, do = case(seed + c + h_q, h_q, h_kv, n * c, n * c, d, dtype)
        lse, delta = torch.zeros(h_q, n * c), torch.zeros(h_q, n * c)
        self.pairs, self.want = _pairs(n, causal), {}
        for qc, kc in self.pairs:
            if only is not None and qc not in only:
                _slices(lse, qc, c).fill_(8.0)       # any will do: these pairs are only in the way
                continue
            x = [np64(_slices(t, i, c)) for t, i in ((q, qc), (k, kc), (v, kc), (do, qc))]
            O, L = A.attention_fwd(*x[:3], self.scale, causal=causal)
            _slices(lse, qc, c).copy_(torch.from_numpy(L))
            _slices(delta, qc, c).copy_(torch.from_numpy(A.delta_rows(O, x[3])))
            self.want[qc, kc] = A.attention_bwd(*x, self.scale, causal=causal)
        self.x = [t.to(dev()) for t in (q, k, v, lse, delta, do)]
        self.out = [torch.full((h, n * c, d), 0.5, device=dev()) for h in (h_q, h_kv, h_kv)]
        # fp32 gradients and those of grouped heads and short causal rows: the bound grows with their magnitude
        self.tol, self.per = TOL[dtype], 4 if dtype == BF16 else 1

    def fresh(self):
        return [torch.full_like(t, 0.5) for t in self.out]

    def check(self, got, acc=lambda qc, kc: (False, False), which=(0, 1, 2)):
        for (qc, kc), want in self.want.items():
            add = acc(qc, kc)
            for i in which:
                g = _slices(got[i], (qc, kc, kc)[i], self.c)
                bound = self.tol * max(1.0, abs(want[i]).max() / self.per)
                assert maxerr(g, want[i] + (0.5 if add[i > 0] else 0.0)) <= bound, (qc, kc, i)

    def chunks(self, got):
        return B.BackwardChunks(*self.x[:3], *self.x[3:], *got, self.c, self.scale)


BWD = [
    # dtype, h_q, h_kv, c, n, causal, several workgroups per key tile
    (BF16, 32, 32, 300, 4, False, False),    # dq by 256-row workgroups
    (BF16, 32, 32, 300, 4, True, False),
    (BF16, 8, 2, 1024, 4, False, True),      # key tiles shared, sums picked up from all four pairs
    (BF16, 8, 2, 700, 4, True, True),        # the same, ragged and causal
    (BF16, 8, 1, 130, 19, False, True),      # more pairs than a launch takes
    (F32, 8, 2, 300, 4, False, True),
    (F32, 12, 1, 260, 3, True, True),
    (F32, 40, 40, 150, 4, False, False),
]


@pytest.mark.parametrize("dtype,h_q,h_kv,c,n,causal,shared", BWD)
def test_backward_lists(dtype, h_q, h_kv, c, n, causal, shared):
    """Gradients overwritten or added to, by pair and side; the other side alone; and no scratch at all."""
    x = _Backward(dtype, h_q, h_kv, c, n, causal)
    bwd = x.chunks(x.out)
    per = min(n, 16)
    assert (bwd.lib.dfa_chunk_bwd_workspace(ctypes.byref(bwd.sh), per, 1, 1) > 0) == shared
    acc = lambda qc, kc: (qc % 2 == 1, qc % 3 == 1)
    bwd.launch([(qc, kc, *acc(qc, kc)) for qc, kc in x.pairs], causal)
    x.check(x.out, acc)
    for side in ((0,), (1, 2)):
        got = x.fresh()
        bwd = x.chunks(got)
        _launch_without(bwd, x, {0, 1, 2} - set(side), 0)
        x.check(got, which=side)
        assert all(bool((got[i] == 0.5).all()) for i in {0, 1, 2} - set(side))
    got = x.fresh()
    _launch_without(x.chunks(got), x, (), 0)
    x.check(got)


def _launch_without(bwd, x, missing, n_bytes, ws=None):
    """The list through the C ABI, without some of the gradients (0: dq, 1: dk, 2: dv), with n_bytes of scratch."""
    sh = bwd.sh
    sh.causal = int(x.causal)
    arr = (B.DfaBwdPair * x.n)()
    for a, (qc, kc) in zip(arr, x.pairs):
        a.q, a.lse, a.delta, a.dO, a.dq = (t[qc] for t in bwd.by_q)
        a.k, a.v, a.dk, a.dv = (t[kc] for t in bwd.by_kv)
        for i in missing:
            setattr(a, ("dq", "dk", "dv")[i], None)
    assert bwd.lib.dfa_chunk_bwd_batch(ctypes.byref(sh), arr, x.n, ws.data_ptr() if n_bytes else None, n_bytes,
                                       torch.cuda.current_stream().cuda_stream) == 0


def test_backward_list_of_many_key_tiles():
    """2816 dk/dv workgroups: two launches of the whole list, one per kind; three of the eight pairs are checked."""
    x = _Backward(BF16, 32, 32, 1300, 8, True, only=(0, 3, 7))
    acc = lambda qc, kc: (qc == 3, qc == 7)
    x.chunks(x.out).launch([(qc, kc, *acc(qc, kc)) for qc, kc in x.pairs], True)
    x.check(x.out, acc)


@pytest.mark.parametrize("dtype,h_q,h_kv,c,n,causal", [(BF16, 8, 1, 300, 1, False), (BF16, 8, 2, 700, 2, True), (F32, 8, 1, 300, 2, False)])
def test_backward_with_any_amount_of_scratch(dtype, h_q, h_kv, c, n, causal):
    """Less scratch than asked for divides the work into fewer parts: the bytes that were given are all that is written,
    the gradients are right, and the same bytes give the same bits."""
    x = _Backward(dtype, h_q, h_kv, c, n, causal)
    lib, sh = dfa.load_library(), x.chunks(x.out).sh
    sh.causal = int(causal)
    full = lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), n, 1, 1)
    assert full > 0
    for n_bytes in (0, 16, full // 4, full // 2 + 16, full - 16, full, full + 4096):
        n_bytes &= ~15
        both = []
        for fill in (0.0, float("nan")):
            ws = torch.full((n_bytes // 4 + 1024,), fill, device=dev())
            ws[n_bytes // 4:] = 7.0
            got = x.fresh()
            _launch_without(x.chunks(got), x, (), n_bytes, ws)
            assert bool((ws[n_bytes // 4:] == 7.0).all())
            both.append(got)
        x.check(both[0])
        assert all(torch.equal(a, b) for a, b in zip(*both))


@pytest.mark.parametrize("dtype,d", [(F32, 64), (F32, 128), (BF16, 128)])
@pytest.mark.parametrize("p,c", [(5, 70), (8, 128)])
def test_schedule_on_position_major_tensors(dtype, d, p, c):
    """q, k, v, dO stored [N, heads, d]: every operand is a strided slice, the outputs are not."""
    h_q, h_kv, n = 4, 2, p * c
    scale = d ** -0.5
    x = case(9600 + n, h_q, h_kv, n, n, d, dtype)
    O, L = A.attention_fwd(*(np64(t) for t in x[:3]), scale)
    want = A.attention_bwd(*(np64(t) for t in x), scale)
    Q, K, V, dO = (t.transpose(0, 1).contiguous().to(dev()).transpose(0, 1) for t in x)
    assert Q.stride() == (d, h_q * d, 1)
    bufs = driver.Buffers(h_q, h_kv, n, d, p, dev())
    driver.run_all_workers(Q, K, V, dO, scale, p, bufs)
    tol = TOL[dtype]
    assert maxerr(bufs.O, O) <= tol and maxerr(bufs.L, L) <= tol
    for got, w in zip((bufs.dQ, bufs.dK, bufs.dV), want):
        assert maxerr(got, w) <= tol * max(1.0, np.abs(w).max() / 4)
