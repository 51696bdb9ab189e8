"""What weights and sums are held in where one call stands in for several pairs (walks, one causal call of all workers): no less than
in the pairs.  Keys of one chunk are made to outweigh all others (their share of a row's sum is e^-40 and less), so that a row's
result is that of one pair, whose precision the others cannot hide."""
import numpy as np
import pytest
import torch

from paper_2310_03294_amd import binding as B, driver
from gpu_util import case, dev, np64
from oracle import attention as A

pytestmark = pytest.mark.gpu

BF16 = torch.bfloat16
SCALE = 128 ** -0.5
# of o where the weights have 16 bits: 2^-17 of a weight, and twice that again for scores, exponentials and sums in fp32 and the merge
# of parts (rounded weights: 1e-3)
REMAINDERS = 3 * 2 ** -17


def _inputs(seed, h_q, h_kv, n, c, heavy):
    """q, k, v of n chunks of c positions; the keys of chunk `heavy` have scores 80 above the others'."""
    q, k, v, _ = case(seed, h_q, h_kv, n * c, n * c, 128, BF16)
    q[..., 0], k[..., 0] = 8.0, 0.0
    k[:, heavy * c:(heavy + 1) * c, 0] = 112.0
    return q, k, v


def _walks(q, k, v, c, walks):
    h_q, n = q.shape[0], q.shape[1]
    O, L = torch.empty(h_q, n, 128, device=dev()), torch.empty(h_q, n, device=dev())
    fwd = B.ForwardChunks(*(t.to(dev()) for t in (q, k, v)), c, SCALE)
    state = fwd.dest(O, L)
    fwd.launch([(qc, kc, state, qc, kc != hi) for qc, lo, hi in walks for kc in range(hi, lo - 1, -1)], None)
    return O, L


def _want(q, k, v, h, rows, lo=0):
    kh = h * k.shape[0] // q.shape[0]
    return A.rows_fwd(np64(q[h, rows]), rows, np64(k[kh, lo:]), np64(v[kh, lo:]), SCALE, lo)


@pytest.mark.parametrize("h_q,h_kv,c,walks", [
    (64, 16, 300, [(2, 0, 2)]),
    (40, 8, 300, [(2, 0, 2), (1, 0, 1)]),
    (64, 64, 1024, [(3, 0, 3)]),
    (64, 16, 1000, [(3, 0, 3)]),
    (16, 4, 4096, [(1, 0, 1)]),
    (64, 16, 1090, [(1, 0, 1), (0, 0, 0)]),
])
def test_row_sums_of_a_walks_own_keys_are_those_of_the_diagonal_pair(h_q, h_kv, c, walks):
    """The diagonal pair alone sums its weights in fp32, as they are: the logsumexp of a few visible keys is off by fp32 rounding of
    the scores (128 products: 2^-24 times 128 times a score of 80 is 6e-4 at the very worst, as a random walk 5e-5), by up to 1e-3
    and more with the rounded weights; rows of few keys have the largest errors."""
    qc = walks[0][0]
    q, k, v = _inputs(310 + c + h_q, h_q, h_kv, qc + 1, c, qc)
    O, L = _walks(q, k, v, c, walks)
    rows = qc * c + np.array([1, 2, 3, 5, 9, 40, 70, c // 2, c - 1])
    for h in (0, h_q // 2, h_q - 1):
        assert np.abs(np64(L[h, rows]) - _want(q, k, v, h, rows)[1]).max() <= 6e-5, h


@pytest.mark.parametrize("h_q,h_kv,c,walks,heavy", [
    (8, 8, 2049, [(3, 0, 3)], 3),                  # 264 workgroups of 64 rows: those of the diagonal pair
    (16, 4, 2048, [(4, 2, 4)], 4),
    (2, 1, 4096, [(i, max(0, i - 1), i) for i in range(4)], 2),
    (32, 8, 100, [(i, max(0, i - 5), i) for i in range(8)], 2),      # the last time step's three pairs
])
def test_walks_keep_the_remainders_that_one_of_their_pairs_has(h_q, h_kv, c, walks, heavy):
    """Relative error of o where a chunk of keys outweighs the others that has weights of 16 bits as a pair of its own or of its
    time step."""
    qc, lo, _ = walks[-1] if len(walks) == 8 else walks[heavy if len(walks) > 1 else 0]
    q, k, v = _inputs(330 + c + h_q, h_q, h_kv, walks[-1][0] + 1, c, heavy)
    O, _ = _walks(q, k, v, c, walks)
    rows = np.arange(qc * c, (qc + 1) * c)
    for h in (0, h_q - 1):
        want = _want(q, k, v, h, rows, lo * c)[0]
        assert np.linalg.norm(np64(O[h, rows]) - want) <= REMAINDERS * np.linalg.norm(want), h


@pytest.mark.parametrize("h_q,h_kv,P,c,mode,qc,heavy", [
    (32, 32, 2, 300, "balanced", 1, 0),            # the one full pair of two workers
    (16, 4, 2, 700, "balanced", 1, 0),
    (16, 4, 4, 300, "balanced", 3, 1),             # the last time step's two pairs
    (32, 8, 8, 100, "balanced", 7, 3),             # ... four
    (32, 8, 8, 500, "ring", 7, 0),                 # ... one
    (32, 8, 8, 100, ("window", 5), 7, 2),          # ... three
])
def test_all_workers_keep_the_remainders_that_a_time_step_has(h_q, h_kv, P, c, mode, qc, heavy):
    q, k, v = _inputs(350 + c + h_q, h_q, h_kv, P, c, heavy)
    bufs = driver.Buffers(h_q, h_kv, P * c, 128, P, dev(), grads=False)
    driver.run_all_workers(*(t.to(dev()) for t in (q, k, v)), None, SCALE, P, bufs, mode=mode, backward=False)
    rows, lo = np.arange(qc * c, (qc + 1) * c), max(0, qc - mode[1]) * c if isinstance(mode, tuple) else 0
    for h in (0, h_q - 1):
        want = _want(q, k, v, h, rows, lo)[0]
        assert np.linalg.norm(np64(bufs.O[h, rows]) - want) <= REMAINDERS * np.linalg.norm(want), h


@pytest.mark.parametrize("d", [64, 128])
def test_f32_gradients_of_one_call_are_no_further_off_than_the_pairs(d):
    """8 workers of 1000 rows: one chain of additions over 8000 rows of dk, dv is 2.3 times as far off as the pairs' (1.6e-6 to 7e-7),
    the sums of 32 rows less far; all against 64 bits."""
    h, P, c = 2, 8, 1000
    n, scale = P * c, d ** -0.5
    q, k, v, do = (t.to(dev()) for t in case(390 + d, h, h, n, n, d, torch.float32))
    want = [torch.empty(h, n, d, dtype=torch.float64, device=dev()) for _ in range(3)]
    hidden = torch.ones(n, n, dtype=torch.bool, device=dev()).triu(1)
    for i in range(h):
        q64, k64, v64, do64 = (t[i].double() for t in (q, k, v, do))
        p = (q64 @ k64.t() * scale).masked_fill_(hidden, -float("inf")).softmax(1)
        dp = do64 @ v64.t()
        ds = p * (dp - (p * dp).sum(1, keepdim=True)) * scale
        want[0][i], want[1][i], want[2][i] = ds @ k64, ds.t() @ q64, p.t() @ do64
    errs = []
    for at_once in (True, False):
        bufs = driver.Buffers(h, h, n, d, P, dev())
        driver.run_all_workers(q, k, v, do, scale, P, bufs, at_once=at_once)
        errs.append([((g.double() - w).norm() / w.norm()).item() for g, w in zip((bufs.dQ, bufs.dK, bufs.dV), want)])
    assert all(a <= 1.05 * b for a, b in zip(*errs)), errs


# (h_q, h_kv, s_q, s_k, d, causal): single rows, blocks of 32 and one row more or less, ragged, both row divisions and shared walks
SPLIT = [(1, 1, 1, 1, 64, False), (2, 1, 31, 33, 64, False), (1, 1, 32, 65, 64, False), (2, 2, 97, 97, 64, True), (32, 8, 300, 300, 64, True),
         (32, 32, 256, 256, 128, False), (32, 8, 333, 301, 128, False), (8, 2, 1024, 1024, 128, True), (32, 32, 513, 511, 128, False)]


def _f32_backward(q, k, v, do, lse, delta, causal):
    grads = [torch.empty_like(t) for t in (q, k, v)]
    B.dfa_chunk_bwd(q, k, v, lse, delta, do, *grads, causal, q.shape[-1] ** -0.5, accumulate=False)
    return grads


@pytest.mark.parametrize("shape", SPLIT, ids=lambda s: "-".join(map(str, s)))
def test_f32_backward_of_split_values(shape):
    """Products of values taken apart into three bf16 ones.  Bound: the exponents, of magnitude up to 16, are rounded to 24 bits (2^-21
    at most, a quarter of it in the mean square), the products' own errors are a fifth of that; fp32 products were 4e-7 to 7.5e-7
    off.  dO of 2^60 and V of 2^-60 (their exponents change, no bit else does) give the same gradients but for those factors;
    an infinite dO is that infinity in the dv of every key that its row sees and touches no other column."""
    h_q, h_kv, s_q, s_k, d, causal = shape
    q, k, v, do = (t.to(dev()) for t in case(4400 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.float32))
    q64, k64, v64, do64 = (t.double() for t in (q, k.repeat_interleave(h_q // h_kv, 0), v.repeat_interleave(h_q // h_kv, 0), do))
    s = q64 @ k64.transpose(1, 2).contiguous() * d ** -0.5
    if causal:
        s = s.masked_fill(torch.ones(s_q, s_k, dtype=torch.bool, device=dev()).triu(1), -float("inf"))
    lse = s.logsumexp(-1).float()
    p = torch.exp(s - lse.double()[..., None])
    dp = do64 @ v64.transpose(1, 2).contiguous()
    delta = (p * dp).sum(-1).float()
    ds = p * (dp - delta.double()[..., None]) * d ** -0.5
    group = lambda t: t.view(h_kv, h_q // h_kv, s_k, d).sum(1)
    want = [ds @ k64, group(ds.transpose(1, 2).contiguous() @ q64), group(p.transpose(1, 2).contiguous() @ do64)]
    got = _f32_backward(q, k, v, do, lse, delta, causal)
    for g, w in zip(got, want):       # (a single key's dS is zero but for rounding)
        assert (g.double() - w).norm().item() <= 2 ** -21 * max(w.norm().item(), 2.0 ** -3 * w.numel() ** 0.5)
    big = 2.0 ** 60
    dq, dk, dv = _f32_backward(q, k, v / big, do * big, lse, delta, causal)
    assert torch.equal(dq, got[0]) and torch.equal(dk, got[1]) and torch.equal(dv, got[2] * big)
    do[:, s_q // 2, 5] = float("inf")
    dv = _f32_backward(q, k, v, do, lse, delta, causal)[2]
    last = s_q // 2 + 1 if causal else s_k
    assert bool((dv[:, :last, 5] == float("inf")).all())
    others = [c for c in range(d) if c != 5]
    assert torch.equal(dv[..., others], got[2][..., others])


@pytest.mark.parametrize("shape", [(1, 1, 200, 256, 64, False), (2, 1, 130, 130, 64, True), (32, 8, 300, 301, 128, False), (8, 8, 2048, 64, 128, False)],
                         ids=lambda s: "-".join(map(str, s)))
def test_f32_backward_of_nan_and_small_values(shape):
    """A NaN stays one whatever its payload, in the operand's rows and columns that it touches and in no other.  dO of 2^-112: of a value
    what lies below 2^-133 is lost, an error of 2^-134 / sqrt(3) each: 2^-22 of dO, and so of dv, 2^-14 at most of P (dP - D), which
    is smaller by P, of the order of 1 / s_k (2^-8)."""
    h_q, h_kv, s_q, s_k, d, causal = shape
    x = [t.to(dev()) for t in case(4500 + s_q + s_k, h_q, h_kv, s_q, s_k, d, torch.float32)]
    q, k, v, do = x
    lse, delta = np.log(s_k) + 0.5 * (q * q).mean(-1), 0.1 * do[..., 0]
    got = _f32_backward(q, k, v, do, lse, delta, causal)
    assert all(bool(g.isfinite().all()) for g in got)
    row, g = s_q // 2, h_q // h_kv
    last = row + 1 if causal else s_k                     # keys that the row sees
    for payload in (0x7f800001, 0x7fc00000, -1):          # signalling with the payload in the lower half, quiet
        bad = do.clone()
        bad.view(torch.int32)[0, row, 5] = payload
        dq, dk, dv = _f32_backward(q, k, v, bad, lse, delta, causal)
        assert bool(dv[0, :last, 5].isnan().all()) and bool(dq[0, row].isnan().all()) and bool(dk[0, :last].isnan().all())
        assert torch.equal(dv[0, :, 6:], got[2][0, :, 6:]) and torch.equal(dq[0, :row], got[0][0, :row])
        assert all(torch.equal(a[1:], b[1:]) for a, b in zip((dk, dv), got[1:])) and torch.equal(dq[1:], got[0][1:])
        bad = k.clone()
        bad.view(torch.int32)[h_kv - 1, 0, 3] = payload
        dq, dk, dv = _f32_backward(q, bad, v, do, lse, delta, causal)
        assert bool(dq[-g:].isnan().all()) and bool(dk[-1, 0].isnan().all()) and bool(dv[-1, 0].isnan().all())
        assert torch.equal(dk[-1, 1:], got[1][-1, 1:]) and torch.equal(dv[-1, 1:], got[2][-1, 1:])
    small = 2.0 ** -112
    tiny = _f32_backward(q, k, v, do * small, lse, delta * small, causal)
    for a, b, bound in zip(tiny, got, (2 ** -14, 2 ** -14, 2 ** -20)):
        assert (a.double() / small - b.double()).norm().item() <= bound * b.double().norm().item()
