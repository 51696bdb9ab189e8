"""GPU parity of walks over several key/value chunks (dfa_span_fwd, dfa_span_bwd) and of merges of several partials in one pass, in
every kernel form they reach; against the fp64 oracle (bounds as in the parity tests)."""
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


def _visible(lo, hi, qc, c):
    """Global index of the last key that each query row of chunk qc sees of the chunks lo .. hi."""
    return qc * c + np.arange(c) if qc == hi else np.full(c, (hi + 1) * c - 1)


# dtype, d, heads, chunk, walks (query chunk, first and last key/value chunk); which of them continue from a state; the form: query
# rows of a workgroup, parts of a tile, parts that the keys are cut in (test_span_host checks that it is the one taken)
FWD = [
    (BF16, 128, 4, 2, 200, [(5, 0, 5), (4, 4, 4), (3, 0, 2), (2, 1, 2)], (1, 3), (64, 4, 6)),
    (BF16, 128, 3, 1, 70, [(1, 0, 1), (0, 0, 0), (2, 0, 0)], (), (64, 4, 1)),          # heads that do not divide into XCDs
    (BF16, 128, 8, 8, 512, [(4, 0, 4)], (), (64, 4, 4)),                               # cut at chunk ends
    (BF16, 128, 8, 2, 128, [(i, max(0, i - 2), i) for i in range(18)], (0, 7), (64, 4, 1)),      # more walks than a launch takes
    (BF16, 128, 40, 8, 300, [(2, 0, 2), (0, 0, 0), (1, 0, 0)], (2,), (64, 4, 1)),
    (BF16, 128, 64, 16, 300, [(2, 0, 2)], (0,), (128, 2, 1)),
    (BF16, 128, 64, 8, 300, [(2, 0, 2), (0, 0, 0), (1, 0, 0)], (2,), (128, 2, 1)),     # with a diagonal alone and no own keys
    (BF16, 128, 40, 8, 600, [(2, 0, 2)], (0,), (128, 2, 1)),
    (BF16, 128, 64, 64, 1024, [(3, 0, 3)], (0,), (256, 1, 1)),                         # whole tiles
    (BF16, 128, 64, 16, 1000, [(3, 0, 3)], (), (256, 1, 1)),                           # ragged
    (BF16, 128, 64, 16, 1280, [(2, 0, 2), (0, 0, 0)], (1,), (256, 1, 1)),              # whole tiles, with a diagonal alone
    (BF16, 128, 64, 64, 1000, [(3, 0, 3), (2, 0, 2), (1, 0, 1), (0, 0, 0)], (2,), (256, 1, 1)),
    (BF16, 128, 8, 2, 2304, [(2, 0, 2)], (0,), (256, 1, 3)),                           # the diagonal pair apart, the keys before it cut
    (BF16, 128, 8, 4, 2200, [(2, 0, 2), (1, 0, 0)], (1,), (256, 1, 2)),                # the same beside a pair
    (BF16, 128, 8, 4, 2100, [(2, 1, 2), (1, 0, 0), (0, 0, 0)], (1,), (128, 2, 1)),     # diagonal and full pairs alone: lists
    (F32, 128, 2, 1, 100, [(4, 0, 4), (1, 1, 1), (3, 0, 2)], (0,), (32, 4, 3)),
    (F32, 64, 3, 3, 70, [(2, 0, 2), (0, 0, 0)], (1,), (32, 4, 1)),
    (F32, 128, 40, 20, 200, [(2, 0, 2), (1, 0, 0), (0, 0, 0)], (1,), (64, 2, 4)),
    (F32, 128, 48, 16, 300, [(2, 0, 2)], (0,), (64, 2, 1)),
    (F32, 64, 48, 16, 300, [(2, 0, 2)], (), (64, 2, 1)),
]


@pytest.mark.parametrize("o_dtype", [F32, BF16])
@pytest.mark.parametrize("dtype,d,h_q,h_kv,c,walks,acc,form", FWD)
def test_forward_walks(dtype, d, h_q, h_kv, c, walks, acc, form, o_dtype):
    """Every second walk's result goes to a buffer of its own; two heads against the oracle."""
    n, scale, tol = max(w[0] for w in walks) + 1, d ** -0.5, 2e-2 if o_dtype == BF16 else TOL[dtype]
    q, k, v, _ = case(700 + c + h_q, h_q, h_kv, n * c, n * c, d, dtype)
    o0, lse0 = (torch.randn(h_q, n * c, d) * 0.1).to(o_dtype), torch.randn(h_q, n * c) + 5
    O, L = o0.to(dev()), lse0.to(dev())
    fwd = B.ForwardChunks(*(t.to(dev()) for t in (q, k, v)), c, scale)
    state, own, pairs = fwd.dest(O, L), {}, []
    for i, (qc, lo, hi) in enumerate(walks):
        dest, chunk = state, qc
        if i % 2 and i not in acc:
            own[i] = (torch.empty(h_q, c, d, dtype=o_dtype, device=dev()), torch.empty(h_q, c, device=dev()))
            dest, chunk = fwd.dest(*own[i]), 0
        pairs += [(qc, kc, dest, chunk, kc != hi or i in acc) for kc in range(hi, lo - 1, -1)]
    fwd.launch(pairs, None)
    for i, (qc, lo, hi) in enumerate(walks):
        rows, keys = slice(qc * c, (qc + 1) * c), slice(lo * c, (hi + 1) * c)
        got_o, got_l = own[i] if i in own else (O[:, rows], L[:, rows])
        for h in (0, h_q - 1):
            kh = h * h_kv // h_q
            want = A.rows_fwd(np64(q[h, rows]), _visible(lo, hi, qc, c), np64(k[kh, keys]), np64(v[kh, keys]), scale, lo * c)
            if i in acc:
                want = A.merge(np64(o0[h, rows])[None], np64(lse0[h, rows])[None], want[0][None], want[1][None])
                want = want[0][0], want[1][0]
            assert maxerr(got_o[h], want[0]) <= tol and maxerr(got_l[h], want[1]) <= TOL[dtype], (i, h)
    used = {w[0] for i, w in enumerate(walks) if i not in own}
    for j in set(range(n)) - used:      # untouched
        assert torch.equal(O[:, j * c:(j + 1) * c].cpu(), o0[:, j * c:(j + 1) * c])


@pytest.mark.parametrize("h_q,h_kv,c,walks", [
    (8, 8, 1000, [(2, 0, 2)]),                     # a worker's walk whose chunk has 128 workgroups of 64 rows
    (8, 2, 2048, [(4, 2, 4)]),                     # ... 256
    (8, 4, 2048, [(0, 0, 0), (1, 0, 1)]),          # two workers, 512 together
    (16, 4, 2048, [(0, 0, 0)]),                    # one worker, 512
])
def test_walks_keep_the_remainders_of_the_weights(h_q, h_kv, c, walks):
    """Where the pairs as calls of their own have weights of 16 bits, so have the walks.  Bound of the relative error: 2^-17 of
    a weight, and twice that again for scores, exponentials and sums in fp32 and the merge of parts (rounded weights: 1e-3)."""
    n, scale = max(w[0] for w in walks) + 1, 128 ** -0.5
    q, k, v, _ = case(900 + c + h_q, h_q, h_kv, n * c, n * c, 128, BF16)
    O, L = torch.empty(h_q, n * c, 128, device=dev()), torch.empty(h_q, n * c, device=dev())
    fwd = B.ForwardChunks(*(t.to(dev()) for t in (q, k, v)), c, scale)
    state = fwd.dest(O, L)
    fwd.launch([(qc, kc, state, qc, kc != hi) for qc, lo, hi in walks for kc in range(hi, lo - 1, -1)], None)
    for qc, lo, hi in walks:
        rows, keys, h = slice(qc * c, (qc + 1) * c), slice(lo * c, (hi + 1) * c), h_q - 1
        want = A.rows_fwd(np64(q[h, rows]), _visible(lo, hi, qc, c), np64(k[h_kv - 1, keys]), np64(v[h_kv - 1, keys]), scale, lo * c)
        assert np.linalg.norm(np64(O[h, rows]) - want[0]) <= 3 * 2 ** -17 * np.linalg.norm(want[0]), qc


@pytest.mark.parametrize("ws", [0, 1, 2])
def test_forward_walk_with_any_scratch(ws):
    """None, half and all of the scratch asked for: nothing is written behind it."""
    h, c, d, n = 4, 200, 128, 6
    q, k, v, _ = case(801, h, h, n * c, n * c, d, BF16)
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    O, L = torch.empty(h, c, d, device=dev()), torch.empty(h, c, device=dev())
    lib, sh = dfa.load_library(), B._make_shape(Q[:, :c], K, False, d ** -0.5, B.DFA_BF16)
    span = B.DfaFwdSpan(Q[:, (n - 1) * c:].data_ptr(), K.data_ptr(), V.data_ptr(), O.data_ptr(), L.data_ptr(), c * d, d, c,
                        n * c, 1, 0, 0)
    sh.q_stride_h = n * c * d
    full = lib.dfa_span_fwd_workspace(ctypes.byref(sh), ctypes.byref(span), 1)
    assert full > 0
    size = (0, full // 2 & ~15, full)[ws]
    buf = torch.full((size // 4 + 1024,), 7.0, device=dev())
    assert lib.dfa_span_fwd(ctypes.byref(sh), ctypes.byref(span), 1, buf.data_ptr() if size else None, size,
                            torch.cuda.current_stream().cuda_stream) == 0
    assert bool((buf[size // 4:] == 7.0).all())
    for h_ in (0, h - 1):
        want = A.rows_fwd(np64(q[h_, (n - 1) * c:]), (n - 1) * c + np.arange(c), np64(k[h_]), np64(v[h_]), d ** -0.5)
        assert maxerr(O[h_], want[0]) <= TOL[BF16] and maxerr(L[h_], want[1]) <= TOL[BF16]


@pytest.mark.parametrize("d,dtype", [(64, F32), (128, F32), (128, BF16)])
@pytest.mark.parametrize("parts", [(2,), (1, 3), (8, 1, 9), (17,), (2,) * 18])
def test_merges_of_several_partials(d, dtype, parts):
    """parts[i] partials into chunk i, in one pass each (more than a launch takes: in several); empty ones among them."""
    h, c = 3, 37
    g = torch.Generator().manual_seed(sum(parts) + d)
    o, lse = torch.randn(h, len(parts) * c, d, generator=g).to(dtype), 3 * torch.randn(h, len(parts) * c, generator=g)
    lse[:, 5] = -np.inf
    O, L, todo, want = o.to(dev()), lse.to(dev()), [], []
    for i, m in enumerate(parts):
        wo, wl = np64(o[:, i * c:(i + 1) * c]), np64(lse[:, i * c:(i + 1) * c])
        for j in range(m):
            po, pl = torch.randn(h, c, d, generator=g).to(dtype), 3 * torch.randn(h, c, generator=g)
            if j == 1:
                po[:, :9], pl[:, :9] = 0, -np.inf
            todo.append((i, po.to(dev()), pl.to(dev())))
            wo, wl = A.merge(wo, wl, np64(po), np64(pl))
        want.append((wo, wl))
    B.dfa_merge_batch(O, L, c, todo)
    for i, (wo, wl) in enumerate(want):
        assert maxerr(O[:, i * c:(i + 1) * c], wo) <= (1e-5 if dtype == F32 else 2e-2)
        assert maxerr(L[:, i * c:(i + 1) * c], wl) <= 1e-5


@pytest.mark.parametrize("d,dtype", [(64, F32), (128, F32), (128, BF16)])
@pytest.mark.parametrize("m", [2, 9])
def test_merges_hand_on_what_is_no_number(d, dtype, m):
    """NaN and infinities come out of several partials in one pass where they come out of one merge after the other."""
    h, c, g = 2, 12, torch.Generator().manual_seed(m)
    nan, inf = float("nan"), float("inf")
    o, lse = torch.randn(h, c, d, generator=g).to(dtype), torch.randn(h, c, generator=g)
    parts = [(torch.randn(h, c, d, generator=g).to(dtype), torch.randn(h, c, generator=g)) for _ in range(m)]
    o[:, 0], lse[:, 0] = nan, -inf                      # a state that is empty and no number
    parts[0][0][:, 1], parts[0][1][:, 1] = nan, -inf    # such a partial
    for x, l in [(o, lse), *parts]:                     # all of them (a query that is no number)
        x[:, 2], l[:, 2] = nan, -inf
    lse[:, 3], parts[1][1][:, 4] = nan, nan
    o[:, 5], parts[0][0][:, 6] = inf, -inf
    o[:, 7], lse[:, 7] = inf, -inf
    for _, l in [(o, lse), *parts]:
        l[:, 8] = -inf                                  # all empty
    parts[m - 1][0][:, 9], parts[m - 1][1][:, 9] = nan, -inf
    for x, l in [(o, lse), *parts[:-1]]:                # all but the last
        x[:, 10], l[:, 10] = nan, -inf
    one, together = ((o.to(dev()), lse.to(dev())) for _ in range(2))
    parts = [(x.to(dev()), l.to(dev())) for x, l in parts]
    for x, l in parts:
        dfa.dfa_merge(*one, x, l)
    B.dfa_merge_batch(*together, c, [(0, x, l) for x, l in parts])
    for a, b in zip(one, together):
        assert torch.equal(a.isnan(), b.isnan()) and torch.equal(a.isinf(), b.isinf())
        finite = a.isfinite()
        # (m roundings of the stored o against one)
        assert (a[finite].float() - b[finite].float()).abs().max().item() <= (1e-5 if dtype == F32 else m * 2 ** -7)


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("acc", [False, True])
def test_cut_walks_hand_on_what_is_no_number(dtype, acc):
    """A query, a key and a value that are no numbers, and an empty state with any o, in a walk whose keys are cut in parts: NaN
    in the rows in which the pairs one after the other have it."""
    h, c, d, n = 2, 64, 128, 12
    q, k, v, _ = case(880, h, h, n * c, n * c, d, dtype)
    q[0, (n - 1) * c + 5] = float("nan")
    k[1, 7, 0] = float("nan")                # (in the last pair: a forward takes the state that it leaves for an empty one)
    v[1, 8 * c + 9, 1] = float("nan")
    o0, lse0 = torch.randn(h, c, d), torch.randn(h, c)
    o0[:, 20], lse0[:, 20] = float("nan"), -float("inf")        # empty: its o is not looked at
    lse0[0, 21] = float("nan")
    fwd = B.ForwardChunks(*(t.to(dev()) for t in (q, k, v)), c, d ** -0.5)
    got = []
    for at_once in (True, False):
        o, lse = o0.to(dev()), lse0.to(dev())
        dest = fwd.dest(o, lse)
        pairs = [(n - 1, kc, dest, 0, acc or kc != n - 1) for kc in range(n - 1, -1, -1)]
        if at_once:
            sh, span = fwd.sh, B.DfaFwdSpan(fwd.q[n - 1], fwd.k[0], fwd.v[0], o.data_ptr(), lse.data_ptr(), c * d, d, c, n * c, 1, acc, 0)
            assert fwd.lib.dfa_span_fwd_workspace(ctypes.byref(sh), ctypes.byref(span), 1) > 0      # (it is cut)
            fwd.launch(pairs, None)
        else:
            for pair in pairs:
                fwd.launch([pair], pair[1] == n - 1)
        got.append((o, lse))
    (o, lse), (want_o, want_lse) = got
    assert torch.equal(o.isnan(), want_o.isnan()) and torch.equal(lse.isnan(), want_lse.isnan())
    assert bool(o[0, 5].isnan().all()) and not bool(o[0, 20].isnan().any())
    for a, b in zip((o, lse), (want_o, want_lse)):
        finite = b.isfinite()
        assert (a[finite] - b[finite]).abs().max().item() <= TOL[dtype]


# dtype, d, heads, chunk, query chunk, first and last key/value chunk, heads that are checked
BWD = [
    (BF16, 128, 8, 8, 130, 6, 0, 6, (0, 7)),        # dq by several workgroups per row block, ragged
    (BF16, 128, 8, 2, 200, 4, 1, 4, (0, 7)),        # key tiles shared, too
    (BF16, 128, 4, 4, 128, 5, 0, 3, (0, 3)),        # none of the chunk's own keys
    (BF16, 128, 2, 1, 64, 8, 0, 8, (0, 1)),
    (BF16, 128, 16, 16, 320, 2, 1, 2, (0, 15)),
    (BF16, 128, 32, 32, 256, 40, 0, 40, (0, 31)),   # more than 2560 key tiles: two launches
    (F32, 64, 4, 2, 100, 4, 0, 4, (0, 3)),
    (F32, 128, 4, 2, 100, 4, 0, 4, (0, 3)),
    (F32, 128, 2, 2, 33, 20, 0, 20, (0, 1)),        # dq's walk shared
    (F32, 64, 8, 1, 150, 3, 1, 2, (0, 7)),
]


@pytest.mark.parametrize("acc", [(False, False), (True, False), (True, True)])
@pytest.mark.parametrize("dtype,d,h_q,h_kv,c,qc,lo,hi,heads", BWD)
def test_backward_span(dtype, d, h_q, h_kv, c, qc, lo, hi, heads, acc):
    """Gradients of one query chunk against the chunks lo .. hi, with the logsumexp and D that these give; neighbours untouched."""
    n, scale, g = qc + 1, d ** -0.5, h_q // h_kv
    q, k, v, do = case(900 + c + h_q, h_q, h_kv, n * c, n * c, d, dtype)
    rows, keys = slice(qc * c, (qc + 1) * c), slice(lo * c, (hi + 1) * c)
    vis = _visible(lo, hi, qc, c)
    lse, delta = torch.full((h_q, n * c), 8.0), torch.zeros(h_q, n * c)
    checked = sorted({h for x in heads for h in range(x // g * g, x // g * g + g)})      # whole groups
    for h in checked:
        o, l = A.rows_fwd(np64(q[h, rows]), vis, np64(k[h // g, keys]), np64(v[h // g, keys]), scale, lo * c)
        lse[h, rows] = torch.from_numpy(l).float()
        delta[h, rows] = torch.from_numpy(A.delta_rows(o, np64(do[h, rows]))).float()
    out = [torch.full((x, n * c, d), 0.5, device=dev()) for x in (h_q, h_kv, h_kv)]
    x = [t.to(dev()) for t in (q, k, v, lse, delta, do)]
    bwd = B.BackwardChunks(*x[:3], *x[3:], *out, c, scale)
    bwd.launch_span(qc, lo, hi, *acc)
    per = 4 if dtype == BF16 else 1

    def check(got, want, add):
        assert maxerr(got, want + (0.5 if add else 0.0)) <= TOL[dtype] * max(1.0, abs(want).max() / per)

    for h in heads:
        args = np64(k[h // g, keys]), np64(v[h // g, keys])
        check(out[0][h, rows], A.rows_dq(np64(q[h, rows]), vis, np64(do[h, rows]), np64(lse[h, rows]), np64(delta[h, rows]), *args,
                                         scale, lo * c), acc[0])
        grads = [A.cols_dkdv(*args, np.arange(lo * c, (hi + 1) * c), np64(q[i, rows]), np64(do[i, rows]), np64(lse[i, rows]),
                             np64(delta[i, rows]), scale, qc * c if qc == hi else n * c) for i in range(h // g * g, h // g * g + g)]
        check(out[1][h // g, keys], sum(a for a, _ in grads), acc[1])
        check(out[2][h // g, keys], sum(b for _, b in grads), acc[1])
    for t, own in zip(out, (rows, keys, keys)):
        rest = torch.ones(n * c, dtype=torch.bool)
        rest[own] = False
        assert bool((t[:, rest] == 0.5).all())


@pytest.mark.parametrize("dtype", [F32, BF16])
@pytest.mark.parametrize("P,c", [(1, 64), (5, 70), (8, 96)])
def test_share_at_hand_equals_step_by_step(dtype, P, c):
    """A worker's share in one walk each way, for every worker (helpers among them), against the same share step by step."""
    h_q, h_kv, n, d = 4, 2, P * c, 128
    q, k, v, do = (t.to(dev()) for t in case(950 + n, h_q, h_kv, n, n, d, dtype))
    scale = d ** -0.5
    whole = driver.Buffers(h_q, h_kv, n, d, P, dev())
    driver.run_all_workers(q, k, v, do, scale, P, whole)
    for w in range(P):
        got = []
        for fused in (True, False):
            bufs = driver.Buffers(h_q, h_kv, n, d, P, dev())
            bufs.O.copy_(whole.O); bufs.L.copy_(whole.L); bufs.delta.copy_(whole.delta)      # of the chunks it helps
            remote = driver.helper_partials_for(q, k, v, scale, P, w, bufs)
            driver.run_worker_share(q, k, v, do, scale, P, w, bufs, remote, fused=fused)
            got.append((bufs.O, bufs.L, bufs.dQ, bufs.dK, bufs.dV))
        for a, b in zip(*got):
            assert (a - b).abs().max().item() <= TOL[dtype] * max(1.0, b.abs().max().item() / 4)


@pytest.mark.parametrize("h_q,h_kv,n,d", [(1, 1, 1000, 64), (4, 4, 800, 128), (2, 1, 1090, 64), (3, 1, 130, 128)])
def test_f32_diagonal_by_several_workgroups_per_row_block(h_q, h_kv, n, d):
    """dq's walks over a diagonal chunk shared by several workgroups; with all the scratch, half of it and none."""
    q, k, v, do = case(970 + n, h_q, h_kv, n, n, d, F32)
    x64, scale = [np64(t) for t in (q, k, v, do)], d ** -0.5
    O, L = A.attention_fwd(*x64[:3], scale)
    want = A.attention_bwd(*x64, scale)
    x = [t.to(dev()) for t in (q, k, v, torch.from_numpy(L).float(), torch.from_numpy(A.delta_rows(O, x64[3])).float(), do)]
    lib, sh = dfa.load_library(), B._bwd_shape(*x, torch.empty_like(x[0]), torch.empty_like(x[1]), torch.empty_like(x[1]), True, scale)
    full = lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, 1, 1)
    assert full > 0
    for size in (full, full // 2 & ~15, 0):
        got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
        ws = torch.full((size // 4 + 1024,), 7.0, device=dev())
        pair = B.DfaBwdPair(*(t.data_ptr() for t in x), *(t.data_ptr() for t in got), 1, 0)
        assert lib.dfa_chunk_bwd_batch(ctypes.byref(sh), ctypes.byref(pair), 1, ws.data_ptr() if size else None, size,
                                       torch.cuda.current_stream().cuda_stream) == 0
        assert bool((ws[size // 4:] == 7.0).all())
        for g, w, add in zip(got, want, (0.5, 0.0, 0.0)):
            assert maxerr(g, w + add) <= TOL[F32] * max(1.0, abs(w).max())
