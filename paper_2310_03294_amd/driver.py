"""Runs DistFlashAttn schedules on one GPU with virtual workers.

Host-side sequencing only: which chunk pair is computed when comes from `dfa_schedule`
(Section 3.2, Algorithm 2), every computation is a call into libdfa.so.  "Sending" a
partial result to another worker is just handing over a buffer, since all P workers live
on the same device here.
"""
from __future__ import annotations

import collections
import functools

import torch

from . import binding as B


class Buffers:
    """Device buffers for one run, allocated once so that timed regions allocate nothing."""

    def __init__(self, h_q, h_kv, n, d, p, device, o_dtype=torch.float32, n_partials=1, grads=True, outputs=True,
                 zero_grads=True):
        c = n // p
        self.c, self.p = c, p
        if outputs:     # False: the caller supplies O and L (a backward from saved tensors)
            self.O = torch.empty((h_q, n, d), dtype=o_dtype, device=device)
            self.L = torch.empty((h_q, n), dtype=torch.float32, device=device)
            self.part_o = [torch.empty((h_q, c, d), dtype=o_dtype, device=device) for _ in range(n_partials)]
            self.part_l = [torch.empty((h_q, c), dtype=torch.float32, device=device) for _ in range(n_partials)]
        if grads:
            self.delta = torch.empty((h_q, n), dtype=torch.float32, device=device)
            new = torch.zeros if zero_grads else torch.empty     # False: a whole pass overwrites every chunk
            self.dQ = new((h_q, n, d), dtype=torch.float32, device=device)
            self.dK = new((h_kv, n, d), dtype=torch.float32, device=device)
            self.dV = new((h_kv, n, d), dtype=torch.float32, device=device)


def _chunk(t, i, c):
    return t[:, i * c:(i + 1) * c]


class KVPrefetcher:
    """Emulates the overlap of Section 3.2 (Eq. 3) on one GPU: the key/value chunk a worker needs at
    step t + 1 is copied into a staging buffer on a second stream while step t computes.  The
    device-to-device copy stands in for the fetch from the peer that owns the chunk; the kernels of
    OWN pairs then read the staged copy, so the dependency (copy before use, use before the buffer is
    overwritten) is the real one.  Both streams have the default priority."""

    def __init__(self, K, V, c):
        self.K, self.V, self.c = K, V, c
        self.stream = torch.cuda.Stream()
        self.buf = [(torch.empty_like(K[:, :c]), torch.empty_like(V[:, :c])) for _ in range(2)]
        self.ev = [torch.cuda.Event(), torch.cuda.Event()]
        self.n = 0

    def fetch(self, kv_chunk):
        """Start copying chunk `kv_chunk` into the next staging slot; returns the slot."""
        slot = self.n & 1
        self.n += 1
        # the slot's previous readers (kernels already queued on the compute stream) come first
        self.stream.wait_stream(torch.cuda.current_stream())
        with torch.cuda.stream(self.stream):
            self.buf[slot][0].copy_(_chunk(self.K, kv_chunk, self.c), non_blocking=True)
            self.buf[slot][1].copy_(_chunk(self.V, kv_chunk, self.c), non_blocking=True)
            self.ev[slot].record()
        return slot

    def get(self, slot):
        torch.cuda.current_stream().wait_event(self.ev[slot])
        return self.buf[slot]


def _own_steps(sched):
    return [st for st in sched if st.kind == B.DFA_STEP_OWN]


def forward_worker(Q, K, V, scale, P, w, bufs: Buffers, remote=None, mode="balanced", fused=True, prefetch=None):
    """Forward share of worker w: its diagonal chunk, its OWN pairs folded into (O_w, L_w),
    the partials that arrive from helpers (`remote`: {helper_id: (o, lse)}) merged at the step
    they arrive, and its HELP pairs computed into fresh partial buffers.
    fused: OWN pairs continue from the state in (O_w, L_w) (dfa_chunk_fwd_acc, the attn(q, k, v,
    o, s) call of Algorithms 1-2); otherwise each is a partial result plus a dfa_merge.
    prefetch: a KVPrefetcher; the key/value chunk of every OWN pair is then staged one step ahead
    on a second stream (fused path only).
    Returns {owner_id: (o_part, lse_part)} for the HELP pairs this worker computed."""
    c = bufs.c
    sent = {}
    o_w, l_w = _chunk(bufs.O, w, c), _chunk(bufs.L, w, c)
    fwd = B.ForwardChunks(Q, K, V, c, scale)
    state = fwd.dest(bufs.O, bufs.L)
    sched = B.dfa_schedule(P, w, mode)
    own = _own_steps(sched) if prefetch is not None else []
    nxt, slot = 0, None
    for st in sched:
        if st.kind == B.DFA_STEP_DIAG:
            if own:
                slot = prefetch.fetch(own[0].kv_chunk); nxt = 1      # copy for step 1 runs under the diagonal pair
            fwd.launch([(w, w, state, w, False)], True)
        elif st.kind == B.DFA_STEP_OWN and fused and prefetch is not None:
            k_s, v_s = prefetch.get(slot)
            if nxt < len(own):
                slot = prefetch.fetch(own[nxt].kv_chunk); nxt += 1   # copy for the next step runs under this pair
            B.dfa_chunk_fwd_acc(_chunk(Q, w, c), k_s, v_s, False, scale, o_w, l_w)
        elif st.kind == B.DFA_STEP_OWN and fused:
            fwd.launch([(w, st.kv_chunk, state, w, True)], False)
        elif st.kind == B.DFA_STEP_OWN:
            po, pl = bufs.part_o[0], bufs.part_l[0]
            fwd.launch([(w, st.kv_chunk, fwd.dest(po, pl), 0, False)], False)
            B.dfa_merge(o_w, l_w, po, pl)
        elif st.kind == B.DFA_STEP_HELP:
            po = torch.empty_like(bufs.part_o[0]); pl = torch.empty_like(bufs.part_l[0])
            fwd.launch([(st.q_chunk, w, fwd.dest(po, pl), 0, False)], False)
            sent[st.send_to] = (po, pl)
        if st.recv_from >= 0 and remote is not None:
            ro, rl = remote[st.recv_from]
            B.dfa_merge(o_w, l_w, ro, rl)
    return sent


def _walk(sched, w, state):
    """The pairs of a worker's own chunk, in the order of its steps, as one walk from the empty state."""
    return [(w, st.kv_chunk, state, w, st.kind == B.DFA_STEP_OWN) for st in sched
            if st.kind in (B.DFA_STEP_DIAG, B.DFA_STEP_OWN)]


def _forward_at_hand(Q, K, V, scale, sched, w, bufs: Buffers, remote):
    """forward_worker for a worker that has all its key/value chunks and all partials at hand: one walk over its own and its
    earlier chunks and its HELP pairs as one launch, the partials merged in one pass.  (Step by step, a
    short chunk's pairs are a chain of launches that each leave most of the device idle.)"""
    fwd = B.ForwardChunks(Q, K, V, bufs.c, scale)
    sent, pairs = {}, _walk(sched, w, fwd.dest(bufs.O, bufs.L))
    for st in sched:
        if st.kind == B.DFA_STEP_HELP:
            po = torch.empty_like(bufs.part_o[0]); pl = torch.empty_like(bufs.part_l[0])
            pairs.append((st.q_chunk, w, fwd.dest(po, pl), 0, False))
            sent[st.send_to] = (po, pl)
    fwd.launch(pairs, None if len(pairs) > 1 else True)      # (its own chunk alone is no sequence of several)
    if remote is not None:
        parts = [remote[st.recv_from] for st in sched if st.recv_from >= 0]
        if len({(o.stride(), l.stride()) for o, l in parts}) == 1:
            B.dfa_merge_batch(bufs.O, bufs.L, bufs.c, [(w, o, l) for o, l in parts])
        else:
            for o, l in parts:
                B.dfa_merge(_chunk(bufs.O, w, bufs.c), _chunk(bufs.L, w, bufs.c), o, l)
    return sent


def new_pass():
    """Bookkeeping of one backward pass: which dQ / dK,dV chunks already hold a contribution.
    The first contribution to a chunk overwrites it (no zero-fill, no read of stale values), the
    later ones accumulate."""
    return {"dq": set(), "dkv": set()}


def backward_worker(Q, K, V, dO, scale, P, w, bufs: Buffers, mode="balanced", with_delta=True, touched=None):
    """Backward of the pairs worker w computed in the forward (same pair -> worker assignment),
    from the final merged O and L of each query chunk; nothing of the forward is re-run.
    For a HELP pair the logsumexp and D of the helped chunk must already be in `bufs`
    (in the distributed setting they travel with that chunk's queries and dO).
    touched: a new_pass() record shared by the calls of one pass; None = always accumulate into
    what the gradient buffers hold."""
    c = bufs.c
    bwd = B.BackwardChunks(Q, K, V, bufs.L, bufs.delta, dO, bufs.dQ, bufs.dK, bufs.dV, c, scale)
    for st in B.dfa_schedule(P, w, mode):
        if st.kind == B.DFA_STEP_IDLE:
            continue
        qc, kc = st.q_chunk, st.kv_chunk
        if with_delta and st.kind == B.DFA_STEP_DIAG:
            B.dfa_delta(_chunk(bufs.O, qc, c), _chunk(dO, qc, c), delta=_chunk(bufs.delta, qc, c))
        bwd.launch([(qc, kc, touched is None or qc in touched["dq"], touched is None or kc in touched["dkv"])],
                   st.kind == B.DFA_STEP_DIAG)
        if touched is not None:
            touched["dq"].add(qc); touched["dkv"].add(kc)


def _backward_at_hand(Q, K, V, dO, scale, sched, w, bufs: Buffers):
    """backward_worker for a worker that has all its key/value chunks at hand, into gradient chunks that hold nothing yet: its
    own and its earlier chunks as one call, then its HELP pairs, all with its own key/value chunk.
    (bf16, long chunks of heads that do not divide into XCDs: pair by pair, each of which fills the device, as the XCD with the
    last key tiles of a walk, half of them behind the diagonal, is done before the others.  us, pairs / walk: 8 over 2 heads, 3 x
    8192 1950 / 2130, 16 over 4, 5 x 6000 3912 / 4065, 4 heads, 3 x 16384 3950 / 4108; 8 over 2, 5 x 6000 2148 / 1971; 8 heads, 5 x 8192
    3464 / 3459, 32 over 8, 5 x 4096 3519 / 3451.)"""
    c = bufs.c
    B.dfa_delta(_chunk(bufs.O, w, c), _chunk(dO, w, c), delta=_chunk(bufs.delta, w, c))
    bwd = B.BackwardChunks(Q, K, V, bufs.L, bufs.delta, dO, bufs.dQ, bufs.dK, bufs.dV, c, scale)
    own = [st.kv_chunk for st in sched if st.kind in (B.DFA_STEP_DIAG, B.DFA_STEP_OWN)]
    if len(own) == 1 or (Q.dtype == torch.bfloat16 and K.shape[0] % 8 and Q.shape[0] * c * c > 3 << 27):
        for kc in own:
            bwd.launch([(w, kc, kc != w, False)], kc == w)
    else:
        bwd.launch_span(w, min(own), w, False, False)
    for st in sched:
        if st.kind == B.DFA_STEP_HELP:
            bwd.launch([(st.q_chunk, w, False, True)], False)


def run_worker_share(Q, K, V, dO, scale, P, w, bufs: Buffers, remote, fused=True):
    """One pass of worker w's whole share: forward (incl. merges of the helpers' partials),
    the D pre-pass and the backward of the same pairs.  The gradient chunks the share touches are
    overwritten with the share's own sums (first contribution overwrites, the rest accumulate).
    fused: all chunks and partials being there, the worker's pairs are one walk each way (a short chunk's step by step: 8 heads x 512,
    P = 8, 183 us, as one walk 74); otherwise step by step."""
    sched = B.dfa_schedule(P, w)
    if fused and _fits_a_call(len(sched) * bufs.c, K, bufs.dK):
        _forward_at_hand(Q, K, V, scale, sched, w, bufs, remote)
        _backward_at_hand(Q, K, V, dO, scale, sched, w, bufs)
        return
    forward_worker(Q, K, V, scale, P, w, bufs, remote=remote, fused=fused)
    backward_worker(Q, K, V, dO, scale, P, w, bufs, touched=new_pass())


def helper_partials_for(Q, K, V, scale, P, w, bufs: Buffers):
    """The partial results other workers compute for worker w's queries under the balanced
    schedule (what arrives over the network in the distributed setting)."""
    c = bufs.c
    out = {}
    for st in B.dfa_schedule(P, w):
        if st.recv_from >= 0:
            h = st.recv_from
            po = torch.empty_like(bufs.part_o[0]); pl = torch.empty_like(bufs.part_l[0])
            B.dfa_chunk_fwd(_chunk(Q, w, c), _chunk(K, h, c), _chunk(V, h, c), False, scale, o=po, lse=pl)
            out[h] = (po, pl)
    return out


def _partials(bufs: Buffers, n):
    """n partial (o, lse) buffers, or as many as there is memory for (at least the first); kept in bufs, so that a later
    pass allocates nothing.  A pass of all workers holds up to (P - 1) / 2 of them, half as much as O."""
    try:
        while len(bufs.part_o) < n:
            part = torch.empty_like(bufs.part_o[0]), torch.empty_like(bufs.part_l[0])
            bufs.part_o.append(part[0]); bufs.part_l.append(part[1])
    except torch.OutOfMemoryError:
        pass
    return list(zip(bufs.part_o, bufs.part_l))[:n]


def delta_all_chunks(O, dO, delta, c, P):
    """D of the P chunks of c rows.  One launch, unless the slices of all chunks together are longer than a call takes
    (a sequence stored [N, heads, d] has heads * d elements between its rows): then as few as that makes it."""
    per = max(1, B.MAX_SLICE // max(O.stride(1), dO.stride(1)) // max(1, c))     # chunks per launch
    if per >= P and P * c == O.shape[1] == delta.shape[1] == dO.shape[1]:
        B.dfa_delta(O, dO, delta=delta)       # (without the slices: 4 us of the host's time)
        return
    for i in range(0, P, per):
        rows = slice(i * c, min(i + per, P) * c)
        B.dfa_delta(O[:, rows], dO[:, rows], delta=delta[:, rows])


def _fits_a_call(rows, *tensors):
    """Whether the first `rows` positions of [heads, seq, d] tensors are no longer a slice than a call takes."""
    return all(rows * t.stride(1) <= B.MAX_SLICE for t in tensors)


@functools.lru_cache(maxsize=64, typed=True)
def _whole_triangle(P, mode):
    """Whether a schedule's pairs are those of every chunk with itself and all earlier ones."""
    return ({(st.q_chunk, st.kv_chunk) for w in range(P) for st in B.dfa_schedule(P, w, mode) if st.kind != B.DFA_STEP_IDLE}
            == {(q, k) for q in range(P) for k in range(q + 1)})


@functools.lru_cache(maxsize=64, typed=True)
def _lists_with_remainders(h_q, h_kv, c, P, mode):
    """Whether the bf16 forward's lists of pairs, time step by time step, multiply V by weights of 16 bits (64-row form): the set of
    what the lists say (they get shorter with the steps: to P / 2 pairs, in the ring schedule to one), and whether the
    sequence as one call does."""
    lists = {(kind == B.DFA_STEP_DIAG, n) for steps in zip(*(B.dfa_schedule(P, w, mode) for w in range(P)))
             for kind, n in collections.Counter(min(st.kind, B.DFA_STEP_OWN) for st in steps if st.kind != B.DFA_STEP_IDLE).items()}
    return ({B.forward_form(h_q, h_kv, c, 128, B.DFA_BF16, causal, n).rows == 64 for causal, n in lists},
            B.sequence_form(h_q, h_kv, P * c, 128, B.DFA_BF16).rows == 64)


def _how_at_once(Q, K, bufs: Buffers, P, mode):
    """(as one causal call, as walks): how the forward of all workers goes out.  (One worker's only pair is that call.)  In
    bf16 neither may hold less of the weights than the lists of pairs do; walks take all in the form of the shortest list,
    which is the slower one for the others of long chunks (ring, us, steps / walks: 32 over 8 heads x 8 x 512 292 / 288,
    16 over 4 x 8 x 700 292 / 263, 8 over 2 x 16 x 1000 879 / 968)."""
    c = bufs.c
    if P == 1:
        return True, True
    if Q.dtype != torch.bfloat16 or c < 1:
        return False, True
    lists, sequence = _lists_with_remainders(Q.shape[0], K.shape[0], c, P, mode)
    one = _whole_triangle(P, mode) and _fits_a_call(P * c, Q, K, bufs.O) and (sequence or True not in lists)
    return one, c <= 768 or len(lists) == 1


def backward_all_workers(Q, K, V, dO, scale, P, bufs: Buffers, mode="balanced", at_once=True):
    """The backward of all P workers' pairs on one device, from the merged O and L and the D of every chunk.
    Where the pairs are those of every chunk with itself and all earlier ones, they are one causal call over the P
    chunks: the sums of a chunk's pairs then stay in registers instead of going through memory pair by pair, and the
    pairs of small chunks, which leave most of the device idle, run side by side.  us in the kernels, time steps / one
    call: 32 over 8 heads x 8192, P = 8, 1960 / 1684; fp32, 4 heads x 8000, P = 8, 2924 / 2318, one head x 1024, P = 4,
    99 / 30.
    Otherwise (at_once False: always) time step by time step: first the pairs of the owners, then those of the helpers.  Each of
    the two groups has every query chunk and every key/value chunk at most once, so its pairs go out as one launch."""
    mode, grads = B.plain_mode(mode), (bufs.dQ, bufs.dK, bufs.dV)
    if at_once and _whole_triangle(P, mode) and _fits_a_call(P * bufs.c, Q, K, *grads):
        bwd = B.BackwardChunks(Q, K, V, bufs.L, bufs.delta, dO, *grads, P * bufs.c, scale)
        bwd.launch([(0, 0, False, False)], None if P > 1 else True)
        return
    touched = new_pass()
    bwd = B.BackwardChunks(Q, K, V, bufs.L, bufs.delta, dO, *grads, bufs.c, scale)
    for steps in zip(*(B.dfa_schedule(P, w, mode) for w in range(P))):
        for kind in (B.DFA_STEP_DIAG, B.DFA_STEP_OWN, B.DFA_STEP_HELP):
            pairs = [(st.q_chunk, st.kv_chunk, st.q_chunk in touched["dq"], st.kv_chunk in touched["dkv"])
                     for st in steps if st.kind == kind]
            assert len({p[0] for p in pairs}) == len({p[1] for p in pairs}) == len(pairs)
            bwd.launch(pairs, kind == B.DFA_STEP_DIAG)
            touched["dq"].update(p[0] for p in pairs)
            touched["dkv"].update(p[1] for p in pairs)


def _forward_step(fwd, state, steps, bufs: Buffers):
    """What all workers compute in one time step, as one launch: the owners' pairs continue from their states, the
    helpers' give partials, which are then "sent" and merged."""
    diag = [st for st in steps if st.kind == B.DFA_STEP_DIAG]
    own = [st for st in steps if st.kind == B.DFA_STEP_OWN]
    helped = [st for st in steps if st.kind == B.DFA_STEP_HELP]
    fwd.launch([(st.q_chunk, st.kv_chunk, state, st.q_chunk, False) for st in diag], True)
    own = [(st.q_chunk, st.kv_chunk, state, st.q_chunk, True) for st in own]
    parts = _partials(bufs, len(helped)) if helped else []
    while own or helped:        # once, unless there are fewer partial buffers than helpers
        now = list(zip(helped, parts))
        fwd.launch(own + [(st.q_chunk, st.kv_chunk, fwd.dest(*part), 0, False) for st, part in now], False)
        B.dfa_merge_batch(bufs.O, bufs.L, bufs.c, [(st.send_to, *part) for st, part in now])
        own, helped = [], helped[len(now):]


def _forward_at_once(fwd, state, scheds, bufs: Buffers):
    """The forward of all workers: every owner's walk over its own and earlier chunks and, as far as there are partial
    buffers (as many as helpers in a time step), the helpers' pairs as one launch, the partials merged; then the helpers'
    pairs that are left."""
    walks = [pair for w, sched in enumerate(scheds) for pair in _walk(sched, w, state)]
    helped = [st for steps in zip(*scheds) for st in steps if st.kind == B.DFA_STEP_HELP]
    parts = _partials(bufs, max(collections.Counter(st.t for st in helped).values())) if helped else []
    while walks or helped:
        now = sorted(zip(helped, parts), key=lambda x: x[0].send_to)      # (the partials of a chunk next to each other)
        fwd.launch(walks + [(st.q_chunk, st.kv_chunk, fwd.dest(*part), 0, False) for st, part in now], None)
        B.dfa_merge_batch(bufs.O, bufs.L, bufs.c, [(st.send_to, *part) for st, part in now])
        walks, helped = [], helped[len(now):]


def run_all_workers(Q, K, V, dO, scale, P, bufs: Buffers, mode="balanced", backward=True, fused=True, at_once=True):
    """The whole schedule of all P workers on one GPU.
    fused: OWN pairs continue from the owner's state instead of partial + merge, and pairs that do not wait for each other go
    out as one launch (a pair of small chunks alone leaves most of one device idle): all of the owners' as one walk
    per owner, or, in bf16 and where the pairs are those of every chunk with itself and all earlier ones, all pairs as one
    causal call (where that is as precise: _how_at_once), which has no partials to write, read and merge (us, forward,
    walks / one call: 32 over 8 heads x 8 x 1024 608 / 503, 8 over 2 x 8 x 2048 596 / 479, 32 x 8 x 300 141 / 72, 8 x 4 x 512
    38 / 32; not in fp32, where the walks cut the keys of the last rows in parts: 8 over 2 heads x 4 x 1024 385 / 478, d = 64,
    2 over 1 x 3 x 700 43 / 74);
    otherwise time step by time step, pair by pair.
    at_once False: the schedule as it is written, fused or not: every pair computed as such at its time step, the partials of the
    helpers written, handed over and merged at theirs, and the backward's pairs in the same order."""
    c, mode = bufs.c, B.plain_mode(mode)
    scheds = [B.dfa_schedule(P, w, mode) for w in range(P)]
    nsteps = len(scheds[0])
    one_call, walks = _how_at_once(Q, K, bufs, P, mode) if fused and at_once else (False, False)
    fwd = B.ForwardChunks(Q, K, V, P * c if one_call else c, scale)
    state = fwd.dest(bufs.O, bufs.L)
    whole = one_call or (walks and _fits_a_call(nsteps * c, K))
    if one_call:
        fwd.launch([(0, 0, state, 0, False)], True if P == 1 else None)
    elif whole:
        _forward_at_once(fwd, state, scheds, bufs)
    for t in range(0 if whole else nsteps):
        steps = [scheds[w][t] for w in range(P)]
        for w, st in enumerate(steps):
            assert st.kind != B.DFA_STEP_HELP or steps[st.send_to].recv_from == w
        if fused:
            _forward_step(fwd, state, steps, bufs)
            continue
        for w, st in enumerate(steps):      # partial + merge, pair by pair
            if st.kind == B.DFA_STEP_DIAG:
                B.dfa_chunk_fwd(_chunk(Q, w, c), _chunk(K, w, c), _chunk(V, w, c), True, scale,
                                o=_chunk(bufs.O, w, c), lse=_chunk(bufs.L, w, c))
            elif st.kind != B.DFA_STEP_IDLE:
                po, pl = bufs.part_o[0], bufs.part_l[0]
                B.dfa_chunk_fwd(_chunk(Q, st.q_chunk, c), _chunk(K, st.kv_chunk, c), _chunk(V, st.kv_chunk, c), False,
                                scale, o=po, lse=pl)
                # HELP: "send", the owner merges it in this same step
                B.dfa_merge(_chunk(bufs.O, st.q_chunk, c), _chunk(bufs.L, st.q_chunk, c), po, pl)
    if backward:
        # a helper's backward needs D of the chunk it helped, so all D vectors come first
        delta_all_chunks(bufs.O, dO, bufs.delta, c, P)
        backward_all_workers(Q, K, V, dO, scale, P, bufs, mode, at_once=fused and at_once)
