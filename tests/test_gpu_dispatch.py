"""GPU parity at the sizes where the launch rules change kernel forms: the smallest calls that reach
each form, with remainders on both axes, against the fp64 oracle (bounds as in the parity tests)."""
import ctypes
import math

import numpy as np
import pytest
import torch

import paper_2310_03294_amd as dfa
from paper_2310_03294_amd import binding as B, driver
from gpu_util import TOL, case, dev, maxerr, np64
from oracle import attention as A
from test_gpu_parity_small import _run_pair

pytestmark = pytest.mark.gpu

# fp32: 1, 2 or 4 parts per tile, chosen by the number of workgroups.  The comment gives the parts of the
# (forward, backward at d = 128).
F32_PARTS = [
    (130, 130, 150, 150, False),   # (2, 1)
    (260, 130, 150, 77, False),    # (1, 1), grouped heads
    (40, 20, 130, 161, False),     # (4, 2), grouped heads
    (40, 40, 130, 161, False),     # (4, 2)
    (520, 520, 130, 130, True),    # (2, 1): causal, 64-row blocks of the forward
    (130, 65, 33, 33, True),       # (2, 2): one row past a block of the forward
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", F32_PARTS)
def test_f32_parts(shape, d):
    h_q, h_kv, s_q, s_k, causal = shape
    _run_pair(torch.float32, h_q, h_kv, s_q, s_k, d, causal)


# bf16 forward: 64-row workgroups with 2 or 4 parts of the keys, 128-row or 256-row workgroups.
FWD_FORMS = [
    # h_q, h_kv, s_q, s_k, causal
    (4, 2, 129, 256, False),      # 64 rows, 2 parts; one row past a block
    (4, 2, 257, 97, False),       # the same, fewer keys than two tiles
    (4, 2, 200, 385, False),      # 64 rows, 4 parts: one key past three tiles
    (2, 2, 65, 31, False),        # fewer keys than one part's block: parts without keys
    (3, 3, 70, 1153, False),
    (96, 32, 190, 300, False),    # 128 rows (288 64-row workgroups)
    (130, 130, 300, 333, False),  # 128 rows: 260 256-row workgroups would leave a last round of 4
    (130, 65, 300, 2111, False),  # the same with 2 parts: more than 2048 keys
    (200, 100, 300, 129, False),  # 256 rows, last round of 144
    (4, 2, 200, 200, True),       # 64 rows, 2 parts
    (4, 2, 450, 450, True),       # 64 rows, 4 parts
    (70, 35, 260, 260, True),     # 128 rows: 210 short workgroups
    (16, 4, 1090, 1090, True),    # 128 rows, 2 parts: 144 workgroups
    (130, 65, 270, 270, True),    # 128 rows: 390
    (96, 32, 129, 33, False),     # 128 rows, 2 parts (288 64-row workgroups): a part with one key
    (88, 44, 140, 31, False),     # the same, the second part without keys
    (90, 45, 161, 161, True),
    (130, 130, 515, 200, False),  # 128 rows: 390 256-row workgroups
]


@pytest.mark.parametrize("shape", FWD_FORMS)
def test_bf16_forward_forms(shape):
    """Forward from the empty state and from the state of another chunk, fp32 and bf16 output."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol = 128, TOL[torch.bfloat16]
    q, k, v, _ = case(5000 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    scale = d ** -0.5
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    O, L = A.attention_fwd(np64(q), np64(k), np64(v), scale, causal=causal)
    for o_dtype in (torch.float32, torch.bfloat16):
        o, lse = dfa.dfa_chunk_fwd(Q, K, V, causal, scale, o_dtype=o_dtype)
        assert maxerr(o, O) <= tol and maxerr(lse, L) <= tol
        if causal:      # its row sums are fp32 sums of the fp32 weights
            assert maxerr(lse, L) <= 1e-4
        # continued from itself: the same o, twice the weight
        dfa.dfa_chunk_fwd_acc(Q, K, V, causal, scale, o, lse)
        assert maxerr(o, O) <= tol and maxerr(lse, L + math.log(2)) <= tol


@pytest.mark.parametrize("h_q,s", [(8, 3300), (22, 6150), (22, 6144)])
def test_bf16_forward_forms_long_causal(h_q, s):
    """64-row workgroups with 4 parts on a long diagonal chunk, 256-row workgroups (ragged and whole tiles)."""
    d, tol = 128, TOL[torch.bfloat16]
    q, k, v, _ = case(6000 + s, h_q, 1, s, s, d, torch.bfloat16)
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    o, lse = dfa.dfa_chunk_fwd(Q, K, V, True, d ** -0.5)
    rows = sorted({0, 1, 31, 32, 63, 64, 65, 255, 256, 257, s // 2, s - 257, s - 65, s - 2, s - 1})
    for h in (0, h_q - 1):
        O, L = A.rows_fwd(np64(q[h, rows]), rows, np64(k[0]), np64(v[0]), d ** -0.5)
        assert maxerr(o[h, rows], O) <= tol and maxerr(lse[h, rows], L) <= 1e-4


@pytest.mark.parametrize("h_q,h_kv,s_q,s_k", [
    (64, 32, 1025, 1100),      # a round of 256-row workgroups and one row more: 64 rows
    (32, 8, 2400, 1025),       # ... and 352 rows of 128
    (48, 48, 1300, 1030),      # a first launch that leaves CUs idle (5 blocks of 48 heads)
    (128, 32, 513, 1153),      # a row of the last round
    (64, 16, 2200, 1090),      # two rounds and the rest
])
def test_bf16_forward_whole_rounds_and_the_rest(h_q, h_kv, s_q, s_k):
    """Rows on both sides of the cut, by samples; outputs with strides of their own, from the empty state and continued."""
    d, tol, scale = 128, TOL[torch.bfloat16], 128 ** -0.5
    q, k, v, _ = case(7000 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    Q = Q.transpose(0, 1).contiguous().transpose(0, 1)            # rows of all heads side by side
    cut = 256 // h_q * 256 * (2 if s_q > 2048 and h_q == 64 else 1)
    rows = sorted({0, 1, 255, 256, cut - 129, cut - 1, cut, min(cut + 63, s_q - 1), min(cut + 129, s_q - 1), s_q - 1})
    for o_dtype in (torch.float32, torch.bfloat16):
        o = torch.full((s_q + 3, h_q, d), 7.0, dtype=o_dtype, device=dev())
        lse = torch.full((h_q, s_q + 5), 7.0, device=dev())
        out = o[:s_q].transpose(0, 1), lse[:, :s_q]
        for weight, f in ((0.0, dfa.dfa_chunk_fwd), (math.log(2), dfa.dfa_chunk_fwd_acc)):
            f(Q, K, V, False, scale, o=out[0], lse=out[1])
            for h in (0, h_q // 2, h_q - 1):
                kv = h * h_kv // h_q
                O, L = A.rows_fwd(np64(q[h, rows]), np.full(len(rows), s_k - 1), np64(k[kv]), np64(v[kv]), scale)
                assert maxerr(out[0][h, rows], O) <= tol and maxerr(out[1][h, rows], L + weight) <= tol
        assert bool((o[s_q:] == 7).all()) and bool((lse[:, s_q:] == 7).all())


WIDE = [(120, 120, 300, 1061, False), (22, 1, 6144, 6144, True)]      # 256-row workgroups, full and diagonal


@pytest.mark.parametrize("shape", WIDE)
def test_bf16_forward_wide_continues(shape):
    """256-row workgroups from a state that another chunk left, with fp32 and bf16 output, by sampled rows."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol = 128, TOL[torch.bfloat16]
    q, k, v, _ = case(6500 + s_q, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    g = torch.Generator().manual_seed(3)
    o0, lse0 = (0.1 * torch.randn(h_q, s_q, d, generator=g)).to(torch.bfloat16), torch.randn(h_q, s_q, generator=g) + 6
    lse0[:, ::5] = -math.inf                 # rows that have seen nothing yet: their o counts for nothing
    rows = sorted({0, 1, 5, 31, 32, 63, 64, 65, 255, 256, 257, s_q // 2, s_q - 44, s_q - 2, s_q - 1})
    for o_dtype in (torch.float32, torch.bfloat16):
        o, lse = o0.to(o_dtype).to(dev()), lse0.to(dev())
        dfa.dfa_chunk_fwd_acc(*(t.to(dev()) for t in (q, k, v)), causal, d ** -0.5, o, lse)
        for h in (0, h_q // 2, h_q - 1):
            kv = h * h_kv // h_q
            want = _sampled(q, k, v, h, kv, rows, d ** -0.5, causal)
            want = A.merge(np64(o0[h, rows]), np64(lse0[h, rows]), *want)
            assert maxerr(o[h, rows], want[0]) <= tol and maxerr(lse[h, rows], want[1]) <= tol


def _sampled(q, k, v, h, kv, rows, scale, causal):
    if causal:
        return A.rows_fwd(np64(q[h, rows]), rows, np64(k[kv]), np64(v[kv]), scale)
    O, L = A.attention_fwd(np64(q[h:h + 1, rows]), np64(k[kv:kv + 1]), np64(v[kv:kv + 1]), scale, causal=False)
    return O[0], L[0]


@pytest.mark.parametrize("top", [150.0, 4000.0])
@pytest.mark.parametrize("shape", WIDE)
def test_bf16_forward_wide_reference_jumps(shape, top):
    """256-row workgroups on scores that jump from one 64-key tile to the next by more than the reference may lag behind
    (2^14 in the exp2 domain): tiles are redone against a moved reference.  Tiles in random order, so that some tower
    over all before them and others lie far below."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol, scale = 128, TOL[torch.bfloat16], 128 ** -0.5
    q, k, v, _ = case(6600 + s_q, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    g = torch.Generator().manual_seed(11)
    u = torch.ones(d) / d ** 0.5
    ramp = torch.linspace(0.0, top, s_k)
    order = torch.randperm((s_k + 63) // 64, generator=g)
    ramp = torch.cat([ramp[i * 64:(i + 1) * 64] for i in order.tolist()]).view(1, s_k, 1)
    q, k = (q + 4.0 * u).to(torch.bfloat16), (0.3 * k + ramp * u).to(torch.bfloat16)
    o, lse = dfa.dfa_chunk_fwd(*(t.to(dev()) for t in (q, k, v)), causal, scale)
    rows = sorted({0, 63, 64, 127, 128, 255, 256, 299, s_q // 3, s_q // 2, s_q - 65, s_q - 1})
    for h in (0, h_q // 2, h_q - 1):
        O, L = _sampled(q, k, v, h, h * h_kv // h_q, rows, scale, causal)
        # lse is formed in fp32 from scores of its own size: 2^-17 of it
        assert maxerr(o[h, rows], O) <= tol and maxerr(lse[h, rows], L) <= max(tol, abs(L).max() * 2.0 ** -17)


@pytest.mark.parametrize("accumulate", [False, True])
@pytest.mark.parametrize("where", ["halves", "second half of the first tile", "one key", "one key of the first tile"])
@pytest.mark.parametrize("shape", WIDE + [(200, 100, 300, 129, False)])
def test_bf16_forward_wide_reference_jumps_inside_a_tile(shape, where, accumulate):
    """The same with jumps at 32 keys, half of a tile: a level of its own for every 32 keys, one half (the first tile's second), one
    key (of which a lane of a diagonal's wavefront has one weight in a sum of eight), from the empty state and from one that lies
    far below the jump and has not seen anything in every fifth row."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol, scale = 128, TOL[torch.bfloat16], 128 ** -0.5
    q, k, v, _ = case(6700 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    g = torch.Generator().manual_seed(12)
    u, level = torch.ones(d) / d ** 0.5, torch.zeros(s_k)
    if where == "halves":
        level = (150 * torch.rand((s_k + 31) // 32, generator=g)).repeat_interleave(32)[:s_k]
    elif where == "second half of the first tile":
        level[32:64] = 150.0
    else:
        level[37 if "first" in where else min(s_k, 1000) // 64 * 64 - 21] = 150.0
    q, k = (q + 4.0 * u).to(torch.bfloat16), (0.3 * k + level.view(1, s_k, 1) * u).to(torch.bfloat16)
    o0, lse0 = 0.1 * torch.randn(h_q, s_q, d, generator=g), torch.randn(h_q, s_q, generator=g) + 6
    lse0[:, ::5] = -math.inf
    o, lse = o0.to(dev()), lse0.to(dev())
    f = dfa.dfa_chunk_fwd_acc if accumulate else dfa.dfa_chunk_fwd
    f(*(t.to(dev()) for t in (q, k, v)), causal, scale, o=o, lse=lse)
    rows = sorted({0, 31, 32, 37, 63, 64, 127, 128, 255, 256, 299, s_q // 3, s_q // 2, s_q - 65, s_q - 1})
    for h in (0, h_q // 2, h_q - 1):
        want = _sampled(q, k, v, h, h * h_kv // h_q, rows, scale, causal)
        if accumulate:
            want = A.merge(np64(o0[h, rows]), np64(lse0[h, rows]), *want)
        assert maxerr(o[h, rows], want[0]) <= tol and maxerr(lse[h, rows], want[1]) <= max(tol, abs(want[1]).max() * 2.0 ** -17)


@pytest.mark.parametrize("key", [5, 40, 63])
def test_bf16_forward_wide_first_reference(key):
    """256-row workgroups: a row's weights are relative to the largest of its first 64, which is 1 and not rounded.  One key has
    e^7.5 times the others' weight; those (e^(x - 7.5) for N(0, 1) scores x, and one in a few hundred rows more than the key's own
    noise allows) are off by 2^-9 / sqrt(3) each, independently: of the sum, (128 keys) 128 e^0.5 e^-7.5 = 0.12 of it times
    1.1e-3 e^0.5 / sqrt(128), 2e-5.  A rounded largest weight alone makes 1.1e-3 of 0.9 of the sum."""
    h_q, h_kv, s_q, s_k, scale = 200, 100, 300, 129, 128 ** -0.5
    q, k, v, _ = case(6800 + key, h_q, h_kv, s_q, s_k, 128, torch.bfloat16)
    q[..., 0], k[..., 0] = 8.0, 0.0
    k[:, key, 0] = 10.625
    sh, form = B.DfaShape(h_q, h_kv, s_q, s_k, 128, B.DFA_BF16, B.DFA_F32, 0, scale), B.DfaForm()
    assert dfa.load_library().dfa_chunk_fwd_form(ctypes.byref(sh), 1, ctypes.byref(form)) == 0 and form.rows == 256
    _, lse = dfa.dfa_chunk_fwd(*(t.to(dev()) for t in (q, k, v)), False, scale)
    _, L = A.attention_fwd(np64(q), np64(k), np64(v), scale, causal=False)
    assert np.sqrt(((np64(lse) - L) ** 2).mean()) <= 8e-5


@pytest.mark.parametrize("shape", [(4, 4, 64, 640, False), (4, 4, 640, 640, True)])
def test_bf16_forward_parts_far_apart(shape):
    """Parts of the keys whose scores differ by hundreds: the other parts' weights underflow."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, scale = 128, 1.0
    q, k, v, _ = case(7000, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    k = (k * torch.linspace(0.01, 4.0, s_k)[None, :, None]).to(torch.bfloat16)      # grows along the keys
    for kk in (k, k.flip(1).contiguous()):
        o, lse = dfa.dfa_chunk_fwd(q.to(dev()), kk.to(dev()), v.to(dev()), causal, scale)
        O, L = A.attention_fwd(np64(q), np64(kk), np64(v), scale, causal=causal)
        # |v| reaches 4.5; a weight is off by 2^-9 of itself
        assert maxerr(o, O) <= 2e-2 and maxerr(lse, L) <= 2e-2 + 2.0 ** -20 * abs(L).max()


@pytest.mark.parametrize("shape", FWD_FORMS)
def test_bf16_forward_infinite_values(shape):
    """A key whose value is infinite gives that infinity to every row that sees it, and NaN where two of them meet; the
    other columns keep their values.  (The key is one that every row sees, and no last one of a ragged chunk.)"""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol, inf = 128, TOL[torch.bfloat16], float("inf")
    q, k, v, _ = case(5500 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    scale = d ** -0.5
    O, L = A.attention_fwd(np64(q), np64(k), np64(v), scale, causal=causal)
    j = 0 if causal else s_k // 2
    v[:, j, 5], v[:, j, 70], v[:, j, 100] = inf, -inf, inf
    if not causal:
        v[:, j + 3, 100] = -inf
    Q, K, V = (t.to(dev()) for t in (q, k, v))
    o, lse = dfa.dfa_chunk_fwd(Q, K, V, causal, scale)
    for again in (False, True):
        if again:
            dfa.dfa_chunk_fwd_acc(Q, K, V, causal, scale, o, lse)
        assert bool((o[..., 5] == inf).all()) and bool((o[..., 70] == -inf).all())
        assert bool((o[..., 100] == inf).all() if causal else o[..., 100].isnan().all())
        rest = [c for c in range(d) if c not in (5, 70, 100)]
        assert maxerr(o[..., rest], O[..., rest]) <= tol and maxerr(lse, L + (math.log(2) if again else 0)) <= tol


# bf16 backward: dq by 128-row workgroups with two key parts or by 256-row ones, next to the dk/dv workgroups.
BWD_FORMS = [
    # h_q, h_kv, s_q, s_k, causal
    (4, 2, 129, 97, False),       # 128 rows, two parts; one row past a block, keys of the last tile in part 0 only
    (3, 3, 70, 161, False),       # the same, one key in the last tile's second part
    (2, 1, 300, 300, True),
    (80, 80, 200, 130, False),    # 256 rows: 160 + 80 workgroups run at once, 160 + 160 would not
    (110, 55, 140, 320, False),   # 128 rows again: 165 + 110 workgroups
    (140, 140, 140, 140, True),   # 256 rows, more than one round, causal
]


@pytest.mark.parametrize("shape", BWD_FORMS)
def test_bf16_backward_forms(shape):
    """All gradients of one call, and dq and dk, dv of calls that want one side, with every mix of overwriting
    and adding."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol = 128, TOL[torch.bfloat16]
    scale = d ** -0.5
    q, k, v, do = case(8000 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    q64, k64, v64, do64 = (np64(t) for t in (q, k, v, do))
    O, L = A.attention_fwd(q64, k64, v64, scale, causal=causal)
    want = A.attention_bwd(q64, k64, v64, do64, scale, causal=causal)
    Q, K, V, dO = (t.to(dev()) for t in (q, k, v, do))
    lse = torch.from_numpy(L).float().to(dev())
    delta = torch.from_numpy(A.delta_rows(O, do64)).float().to(dev())
    # gradients of the short causal rows and sums over a group are larger than those of long chunks
    bound = [tol * max(1.0, abs(w).max() / 4) for w in want]
    for acc_q, acc_kv in ((False, False), (True, False), (False, True), (True, True)):
        got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
        dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, *got, causal, scale, accumulate=acc_q, accumulate_dkv=acc_kv)
        for g, w, b, a in zip(got, want, bound, (acc_q, acc_kv, acc_kv)):
            assert maxerr(g, w + (0.5 if a else 0.0)) <= b
    dq = dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, torch.empty_like(got[0]), None, None, causal, scale)[0]
    _, dk, dv = dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, None, *(torch.empty_like(g) for g in got[1:]), causal, scale)
    for g, w, b in zip((dq, dk, dv), want, bound):
        assert maxerr(g, w) <= b


# dk, dv by several workgroups per key tile: (heads, rows, keys, causal).
BWD_PARTS = [
    (3, 1, 129, 70, False),       # 3 parts, one head each
    (8, 1, 260, 300, False),      # 8 parts, remainders on both axes
    (12, 2, 300, 130, False),     # parts that cut through heads
    (8, 1, 700, 700, True),       # the last key tiles have few query tiles
    (16, 1, 40, 40, True),        # more parts than a tile has heads to give, or as many
]


@pytest.mark.parametrize("shape", BWD_PARTS)
def test_bf16_backward_parts(shape):
    """Against the oracle, and against the same call without scratch (one workgroup per key tile)."""
    h_q, h_kv, s_q, s_k, causal = shape
    d, tol = 128, TOL[torch.bfloat16]
    scale = d ** -0.5
    q, k, v, do = case(9000 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.bfloat16)
    q64, k64, v64, do64 = (np64(t) for t in (q, k, v, do))
    O, L = A.attention_fwd(q64, k64, v64, scale, causal=causal)
    want = A.attention_bwd(q64, k64, v64, do64, scale, causal=causal)
    bound = [tol * max(1.0, abs(w).max() / 4) for w in want]
    Q, K, V, dO = (t.to(dev()) for t in (q, k, v, do))
    lse = torch.from_numpy(L).float().to(dev())
    delta = torch.from_numpy(A.delta_rows(O, do64)).float().to(dev())
    lib = B.load_library()
    for want_dq in (True, False):
        for acc in (False, True):
            got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
            alone = [g.clone() for g in got]
            dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, got[0] if want_dq else None, got[1], got[2], causal, scale,
                              accumulate=acc)
            sh = B._bwd_shape(Q, K, V, lse, delta, dO, alone[0], alone[1], alone[2], causal, scale)
            assert lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, want_dq, 1) > 0
            pair = B.DfaBwdPair(Q.data_ptr(), K.data_ptr(), V.data_ptr(), lse.data_ptr(), delta.data_ptr(),
                                dO.data_ptr(), alone[0].data_ptr() if want_dq else None, alone[1].data_ptr(),
                                alone[2].data_ptr(), acc, acc)
            assert lib.dfa_chunk_bwd_batch(ctypes.byref(sh), ctypes.byref(pair), 1, None, 0,
                                           torch.cuda.current_stream().cuda_stream) == 0
            for i in (0, 1, 2) if want_dq else (1, 2):
                assert maxerr(got[i], want[i] + (0.5 if acc else 0.0)) <= bound[i]
                # the same products, summed in another order in fp32
                assert (got[i] - alone[i]).abs().max().item() <= 1e-5 * max(1.0, abs(want[i]).max())


@pytest.mark.parametrize("h,s_q,s_k,causal", [(1, 1000, 700, False), (1, 1300, 1300, True), (2, 1920, 65, False)])
def test_bf16_backward_parts_of_one_head(h, s_q, s_k, causal):
    """dk, dv of heads of their own by several workgroups per key tile, whose shares are ranges of one head's query tiles."""
    d, tol, scale = 128, TOL[torch.bfloat16], 128 ** -0.5
    q, k, v, do = case(9200 + s_q, h, h, s_q, s_k, d, torch.bfloat16)
    x64 = [np64(t) for t in (q, k, v, do)]
    O, L = A.attention_fwd(*x64[:3], scale, causal=causal)
    want = A.attention_bwd(*x64, scale, causal=causal)
    x = [t.to(dev()) for t in (q, k, v, torch.from_numpy(L).float(), torch.from_numpy(A.delta_rows(O, x64[3])).float(), do)]
    sh, form = B._bwd_shape(*x, torch.empty(h, s_q, d, device=dev()), *(torch.empty(h, s_k, d, device=dev()) for _ in range(2)), causal, scale), B.DfaForm()
    assert B.load_library().dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, 128 << 20, ctypes.byref(form)) == 0 and form.cuts > 1
    for acc in (False, True):
        got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
        dfa.dfa_chunk_bwd(*x, *got, causal, scale, accumulate=acc)
        for g, w in zip(got, want):
            assert maxerr(g, w + (0.5 if acc else 0.0)) <= tol * max(1.0, abs(w).max() / 4)


@pytest.mark.parametrize("h_q,h_kv,s_q,s_k,n,rows", [
    (64, 16, 1000, 8201, 1, 256), (64, 64, 512, 8192, 2, 256), (64, 16, 500, 8199, 2, 256),      # whole rounds of 256-row workgroups
    (64, 16, 1100, 8201, 1, 128), (64, 16, 500, 8191, 2, 128),                                   # a round and a few more; a key too few
])
def test_bf16_dq_alone_forms(h_q, h_kv, s_q, s_k, n, rows):
    """dq alone of one pair and of lists, 256 and 128 rows, by sampled rows; overwriting and adding; nothing written past the rows."""
    d, tol, scale = 128, TOL[torch.bfloat16], 128 ** -0.5
    g = torch.Generator(device=dev()).manual_seed(s_q + s_k)
    rand = lambda *shape: torch.randn(shape, generator=g, device=dev()).to(torch.bfloat16)
    at = sorted({0, 1, 31, 32, 63, 64, 127, 128, 255, 256, s_q // 2, s_q - 1})
    ops, outs, pairs = [], [], (B.DfaBwdPair * n)()
    for i in range(n):
        q, do, k, v = rand(h_q, s_q, d), rand(h_q, s_q, d), rand(h_kv, s_k, d), rand(h_kv, s_k, d)
        lse = math.log(s_k) + 0.5 * (q.float() ** 2).mean(-1)                 # what N(0, 1) keys give a row
        delta = 0.1 * torch.randn(h_q, s_q, generator=g, device=dev())
        ops.append((q, do, k, v, lse, delta))
        outs.append(torch.full((h_q, s_q + 1, d), 0.5, device=dev()))
        pairs[i] = B.DfaBwdPair(q.data_ptr(), k.data_ptr(), v.data_ptr(), lse.data_ptr(), delta.data_ptr(), do.data_ptr(), outs[i].data_ptr(), None, None, i % 2, 0)
    sh, form, lib = B._make_shape(ops[0][0], ops[0][2], False, scale, B.DFA_BF16, lse=ops[0][4], dq=outs[0][:, :s_q], dkv=outs[0]), B.DfaForm(), B.load_library()
    assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), n, 1, 0, 0, ctypes.byref(form)) == 0 and form.rows == rows
    assert lib.dfa_chunk_bwd_batch(ctypes.byref(sh), pairs, n, None, 0, torch.cuda.current_stream().cuda_stream) == 0
    for i, (q, do, k, v, lse, delta) in enumerate(ops):
        for h in (0, h_q // 2, h_q - 1):
            kh = h * h_kv // h_q
            want = A.rows_dq(np64(q[h, at]), np.full(len(at), s_k - 1), np64(do[h, at]), np64(lse[h, at]), np64(delta[h, at]), np64(k[kh]), np64(v[kh]), scale)
            assert maxerr(outs[i][h, at], want + (0.5 if i % 2 else 0.0)) <= 0.02 * abs(want).max()
        assert bool((outs[i][:, s_q] == 0.5).all())


@pytest.mark.parametrize("dtype,d", [(torch.float32, 64), (torch.float32, 128), (torch.bfloat16, 128)])
@pytest.mark.parametrize("p,c", [(19, 24), (5, 70), (2, 130)])
@pytest.mark.parametrize("at_once", [False, True])
def test_schedule_in_batches(dtype, d, p, c, at_once):
    """All workers' pairs of a time step in one launch: more pairs than one launch takes (19 diagonal chunks), ragged
    chunks, operands that are slices with strides of their own; a second pass over the same buffers.  at_once: the walks or the one
    call that stand for them."""
    h_q, h_kv, n = 4, 2, p * c
    scale = d ** -0.5
    q, k, v, do = case(9500 + n, h_q, h_kv, n, n, d, dtype)
    O, L = A.attention_fwd(np64(q), np64(k), np64(v), scale)
    want = A.attention_bwd(np64(q), np64(k), np64(v), np64(do), scale)

    def inside(t):      # an interior slice of a larger tensor
        big = torch.zeros(t.shape[0] + 1, t.shape[1] + 8, d + 8, dtype=t.dtype, device=dev())
        s = big[:t.shape[0], 8:8 + t.shape[1], :d]
        return s.copy_(t.to(dev()))

    Q, K, V, dO = (inside(t) for t in (q, k, v, do))
    bufs = driver.Buffers(h_q, h_kv, n, d, p, dev())
    tol = TOL[dtype]
    for _ in range(2):
        driver.run_all_workers(Q, K, V, dO, scale, p, bufs, at_once=at_once)
        assert maxerr(bufs.O, O) <= tol and maxerr(bufs.L, L) <= tol
        for got, w in zip((bufs.dQ, bufs.dK, bufs.dV), want):
            assert maxerr(got, w) <= tol * max(1.0, abs(w).max() / 4)


# fp32 dk, dv by several workgroups per row block: (heads, rows, keys, causal).
F32_SHARES = [
    (8, 2, 300, 260, False),      # remainders on both axes
    (8, 1, 130, 70, False),
    (12, 1, 700, 700, True),      # more shares than the last row blocks have query tiles
    (6, 2, 1100, 150, False),     # shares that cut through heads
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", F32_SHARES)
def test_f32_backward_shares(shape, d):
    """Against the oracle, overwriting and adding, with and without dq."""
    h_q, h_kv, s_q, s_k, causal = shape
    scale = d ** -0.5
    q, k, v, do = case(9700 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.float32)
    q64, k64, v64, do64 = (np64(t) for t in (q, k, v, do))
    O, L = A.attention_fwd(q64, k64, v64, scale, causal=causal)
    want = A.attention_bwd(q64, k64, v64, do64, scale, causal=causal)
    # fp32 gradients: the bound grows with their magnitude
    bound = [TOL[torch.float32] * max(1.0, abs(w).max()) for w in want]
    Q, K, V, dO = (t.to(dev()) for t in (q, k, v, do))
    lse = torch.from_numpy(L).float().to(dev())
    delta = torch.from_numpy(A.delta_rows(O, do64)).float().to(dev())
    sh = B._bwd_shape(Q, K, V, lse, delta, dO, None, K, V, causal, scale)
    for want_dq in (True, False):
        assert B.load_library().dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, want_dq, 1) > 0
        for acc in (False, True):
            got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
            dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, got[0] if want_dq else None, got[1], got[2], causal, scale,
                              accumulate=acc)
            for i in (0, 1, 2) if want_dq else (1, 2):
                assert maxerr(got[i], want[i] + (0.5 if acc else 0.0)) <= bound[i]


# fp32 backward at d = 128: parts of a tile, shares of the walks of dk, dv and of dq
F32_BWD_FORMS = [
    (4, 1, 97, 97, True, (4, 6, 1)),
    (8, 2, 200, 200, True, (4, 8, 2)),
    (1, 1, 70, 145, False, (2, 1, 1)),
    (1, 1, 300, 300, False, (2, 2, 1)),
    (2, 1, 130, 130, True, None),
    (1, 1, 161, 161, True, (2, 3, 2)),
    (16, 4, 333, 333, True, (1, 12, 2)),
    (32, 8, 300, 300, True, (1, 6, 1)),
    (8, 2, 161, 327, False, None),
]


@pytest.mark.parametrize("h_q,h_kv,s_q,s_k,causal,form", F32_BWD_FORMS)
def test_f32_backward_forms(h_q, h_kv, s_q, s_k, causal, form):
    """Against the oracle, with all scratch and with none (1, 2 and 4 parts undivided), overwriting and adding."""
    d, lib = 128, B.load_library()
    scale = d ** -0.5
    x = case(9950 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.float32)
    x64 = [np64(t) for t in x]
    O, L = A.attention_fwd(*x64[:3], scale, causal=causal)
    want = A.attention_bwd(*x64, scale, causal=causal)
    q, k, v, do = (t.to(dev()) for t in x)
    lse, delta = torch.from_numpy(L).float().to(dev()), torch.from_numpy(A.delta_rows(O, x64[3])).float().to(dev())
    sh = B._make_shape(q, k, causal, scale, B.DFA_F32, lse=lse, dq=q, dkv=k)
    got_form = B.DfaForm()
    assert lib.dfa_chunk_bwd_form(ctypes.byref(sh), 1, 1, 1, 128 << 20, ctypes.byref(got_form)) == 0
    assert form is None or (got_form.parts, got_form.cuts, got_form.q_cuts) == form
    n = lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), 1, 1, 1)
    stream = torch.cuda.current_stream().cuda_stream
    for n_bytes, acc in ((n, False), (n, True), (0, False), (0, True)):
        ws = torch.full((n_bytes // 4 + 256,), 7.0, device=dev())
        got = [torch.full(w.shape, 0.5, device=dev()) for w in want]
        pair = B.DfaBwdPair(*(t.data_ptr() for t in (q, k, v, lse, delta, do, *got)), acc, acc)
        assert lib.dfa_chunk_bwd_batch(ctypes.byref(sh), ctypes.byref(pair), 1, ws.data_ptr() if n_bytes else None, n_bytes, stream) == 0
        assert bool((ws[n_bytes // 4:] == 7.0).all())
        for g, w in zip(got, want):
            bound = TOL[torch.float32] * max(1.0, abs(w).max())      # grows with the magnitude of the sums
            assert maxerr(g, w + (0.5 if acc else 0.0)) <= bound


# fp32 dq by several workgroups per row block, from eight keys per query row on: (heads, rows, keys, pairs)
F32_Q_SHARES = [
    (2, 1, 20, 1000, 1),
    (8, 2, 33, 2500, 1),          # two row blocks
    (16, 1, 60, 1500, 1),         # dk, dv shared too
    (1, 1, 5, 400, 18),           # more pairs than a launch takes
    (4, 4, 100, 801, 2),
    (1, 1, 31, 16384, 1),
]


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("shape", F32_Q_SHARES)
def test_f32_backward_query_shares(shape, d):
    """A list of pairs with all the scratch asked for, half of it and none: against the oracle, overwriting and adding, with
    all gradients and dq alone; nothing is written behind the scratch."""
    h_q, h_kv, s_q, s_k, n = shape
    scale, lib = d ** -0.5, B.load_library()
    ops, want, pairs = [], [], (B.DfaBwdPair * n)()
    for i in range(n):
        x = case(9800 + 31 * i + s_k, h_q, h_kv, s_q, s_k, d, torch.float32)
        x64 = [np64(t) for t in x]
        O, L = A.attention_fwd(*x64[:3], scale, causal=False)
        want.append(A.attention_bwd(*x64, scale, causal=False))
        q, k, v, do = (t.to(dev()) for t in x)
        ops.append((q, k, v, torch.from_numpy(L).float().to(dev()), torch.from_numpy(A.delta_rows(O, x64[3])).float().to(dev()), do))
    sh = B._make_shape(ops[0][0], ops[0][1], False, scale, B.DFA_F32, lse=ops[0][3], dq=ops[0][0], dkv=ops[0][1])
    stream = torch.cuda.current_stream().cuda_stream
    for want_kv in (True, False):
        full = lib.dfa_chunk_bwd_workspace(ctypes.byref(sh), n, 1, want_kv)
        assert full > 0
        for n_bytes, acc in ((full, False), (full, True), (full // 2 & ~15, False), (0, True)):
            ws = torch.full((n_bytes // 4 + 256,), 7.0, device=dev())
            outs = [[torch.full(w.shape, 0.5, device=dev()) for w in ws_i] for ws_i in want]
            for p, o, g in zip(pairs, ops, outs):
                p.q, p.k, p.v, p.lse, p.delta, p.dO = (t.data_ptr() for t in o)
                p.dq, p.dk, p.dv = g[0].data_ptr(), *(t.data_ptr() if want_kv else None for t in g[1:])
                p.accumulate_dq = p.accumulate_dkv = acc
            assert lib.dfa_chunk_bwd_batch(ctypes.byref(sh), pairs, n, ws.data_ptr() if n_bytes else None, n_bytes, stream) == 0
            assert bool((ws[n_bytes // 4:] == 7.0).all())
            for g, w in zip(outs, want):
                for j in range(3 if want_kv else 1):
                    bound = TOL[torch.float32] * max(1.0, abs(w[j]).max())      # grows with the magnitude of the sums
                    assert maxerr(g[j], w[j] + (0.5 if acc else 0.0)) <= bound
                assert want_kv or all(bool((t == 0.5).all()) for t in g[1:])


def test_f32_dq_of_a_long_walk():
    """dq over 16384 keys, from the exact logsumexp and D.  A rounding is off by 2^-24 / sqrt(3) = 3.4e-8 (rms) of the partial
    sum that it rounds, which over a chain of n steps of like size makes 3.4e-8 sqrt(n / 2) of the sum.  Scores and dP (64
    steps each), the exponential and the factors make about 5e-7 of every term, and so of the sum; a wavefront's 4096 keys
    in one chain of 2048 steps would add 1.1e-6, sums of 64 keys each (32 steps, then 64 more) add 2.5e-7.  The bound lies
    between the two totals."""
    h_q, h_kv, s_q, s_k, d = 2, 1, 300, 16384, 128
    scale = d ** -0.5
    q, k, v, do = case(9900, h_q, h_kv, s_q, s_k, d, torch.float32)
    x64 = [np64(t) for t in (q, k, v, do)]
    O, L = A.attention_fwd(*x64[:3], scale, causal=False)
    want = A.attention_bwd(*x64, scale, causal=False)[0]
    Q, K, V, dO = (t.to(dev()) for t in (q, k, v, do))
    lse = torch.from_numpy(L).float().to(dev())
    delta = torch.from_numpy(A.delta_rows(O, x64[3])).float().to(dev())
    dq = dfa.dfa_chunk_bwd(Q, K, V, lse, delta, dO, torch.empty_like(Q), None, None, False, scale)[0]
    assert np.linalg.norm(np64(dq) - want) <= 9e-7 * np.linalg.norm(want)


# One row per lane, and two (from 2049 workgroups of one row per lane on), with remainders.
@pytest.mark.parametrize("o_dtype,heads,rows,d", [
    (torch.float32, 3, 37, 128), (torch.float32, 40, 515, 128), (torch.float32, 64, 1031, 64),
    (torch.bfloat16, 5, 70, 64), (torch.bfloat16, 64, 529, 128), (torch.bfloat16, 20, 4101, 64),
])
def test_merge_rows(o_dtype, heads, rows, d):
    g = torch.Generator().manual_seed(rows)
    oa, ob = (torch.randn(heads, rows, d, generator=g).to(o_dtype) for _ in range(2))
    la, lb = (torch.randn(heads, rows, generator=g) for _ in range(2))
    la[:, ::7], lb[:, ::5] = -math.inf, -math.inf
    O, L = A.merge(np64(oa), np64(la), np64(ob), np64(lb))
    o, lse = oa.to(dev()), la.to(dev())
    dfa.dfa_merge(o, lse, ob.to(dev()), lb.to(dev()))
    # one rounding of a value below 8 to bf16 (2^-6), or a few of fp32
    assert maxerr(o, O) <= (2.0 ** -6 if o_dtype == torch.bfloat16 else 4e-6)
    both = np.isfinite(L)
    assert maxerr(lse[torch.from_numpy(both).to(dev())], L[both]) <= 1e-6 and bool((lse.cpu()[torch.from_numpy(~both)] == -math.inf).all())
