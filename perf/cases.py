"""The calls whose speed counts, over the sizes this library is used at.

A program that trains with DistFlashAttn makes these calls: the chunk kernels through the C ABI's
binding (forward of a diagonal or an earlier key/value chunk, continuing from a state or not, merge,
D, backward), one worker's whole share of the balanced schedule, the schedule of all workers on one
device, and the autograd function around it.  Head counts are those of a 32-head model with 32 or 8
key/value heads, whole or divided over 4 tensor-parallel ranks; chunks run from a few hundred tokens
(short fine-tuning sequences) to 65536 (512K tokens over 8 workers).  bf16 at d = 128 is what training
uses; fp32 at d = 64 and 128 is the precision-reference mode.  Values are i.i.d. N(0, 1), the
workload of the parity configurations.
"""
from __future__ import annotations

import math

import torch

import paper_2310_03294_amd as dfa
from paper_2310_03294_amd import autograd, driver

DEV = "cuda:0"
DTYPES = {"bf16": torch.bfloat16, "f32": torch.float32}


def listed():
    return [
        # The smallest configuration: precision-reference mode, one head, four workers, forward and
        # backward.  Latency and launches count.
        {"name": "schedule_f32_h1_d64_n1k", "kind": "schedule", "h_q": 1, "h_kv": 1, "d": 64, "p": 4, "c": 256,
         "dtype": "f32"},
        # A gradient check of a layer in fp32 at the model's head dimension, grouped heads.
        {"name": "schedule_f32_h8_d128_n4k", "kind": "schedule", "h_q": 8, "h_kv": 2, "d": 128, "p": 4, "c": 1024,
         "dtype": "f32"},
        # A short sequence on a tensor-parallel slice of the heads: a worker's share of small kernels.
        {"name": "share_h8_c512", "kind": "share", "h_q": 8, "h_kv": 8, "p": 8, "c": 512},
        # The heaviest worker's training step at 32K tokens: 5 pairs forward and backward, 3 merges.
        {"name": "share_h32_c4096", "kind": "share", "h_q": 32, "h_kv": 32, "p": 8, "c": 4096},
        # The same with grouped heads at 256K tokens over 16 workers (9 pairs): the largest call.
        {"name": "share_gqa_c16384", "kind": "share", "h_q": 32, "h_kv": 8, "p": 16, "c": 16384},
        # A worker's own (causal) chunk, first step of every schedule, 128K tokens over 8 workers.
        {"name": "fwd_diag_c16384", "kind": "fwd", "h_q": 32, "h_kv": 32, "s_q": 16384, "s_k": 16384, "causal": True,
         "acc": False, "o": "f32"},
        # An earlier chunk folded into the running state, 512K tokens over 8 workers.
        {"name": "fwd_acc_c65536", "kind": "fwd", "h_q": 32, "h_kv": 32, "s_q": 65536, "s_k": 65536, "causal": False,
         "acc": True, "o": "f32"},
        # A helper's partial on ragged chunks of grouped heads, sent as bf16.
        {"name": "fwd_gqa_ragged", "kind": "fwd", "h_q": 32, "h_kv": 8, "s_q": 2777, "s_k": 3001, "causal": False,
         "acc": False, "o": "bf16"},
        # Backward of an earlier chunk, gradients added to what the worker holds, 128K tokens.
        {"name": "bwd_c16384", "kind": "bwd", "h_q": 32, "h_kv": 32, "s_q": 16384, "s_k": 16384, "causal": False,
         "accumulate": True},
        # Backward of a short ragged diagonal chunk with grouped heads.
        {"name": "bwd_gqa_ragged_diag", "kind": "bwd", "h_q": 32, "h_kv": 8, "s_q": 1500, "s_k": 1500, "causal": True,
         "accumulate": False},
        # What follows the attention of a chunk: a helper's partial merged in, then D for the backward.
        {"name": "merge_delta_c16384", "kind": "rows", "h_q": 32, "h_kv": 32, "s_q": 16384, "d": 128, "o": "f32",
         "dtype": "bf16"},
        # One attention layer of a training step through autograd, all workers on one device, with the
        # checkpoint at the attention output.
        {"name": "autograd_gqa_n8k", "kind": "autograd", "h_q": 32, "h_kv": 8, "p": 8, "c": 1024},
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["schedule", "share", "share", "fwd", "fwd", "fwd", "bwd", "bwd", "bwd", "rows", "autograd"])
    h_q, h_kv = rng.choice([(32, 32), (32, 8), (8, 8), (8, 2), (16, 4)])
    if kind == "schedule":      # fp32: small problems
        d = rng.choice([64, 128])
        h_q, h_kv = rng.choice([(1, 1), (2, 1), (4, 4), (8, 2)])
        return {"kind": kind, "h_q": h_q, "h_kv": h_kv, "d": d, "p": rng.choice([2, 3, 4, 8]),
                "c": _log_int(rng, 64, 1024), "dtype": "f32"}
    if kind == "share":
        p = rng.choice([4, 5, 8, 16])
        return {"kind": kind, "h_q": h_q, "h_kv": h_kv, "p": p, "c": _log_int(rng, 256, 12000)}
    if kind == "autograd":
        return {"kind": kind, "h_q": h_q, "h_kv": h_kv, "p": rng.choice([1, 2, 4, 8]), "c": _log_int(rng, 256, 2048)}
    if kind == "rows":
        return {"kind": kind, "h_q": h_q, "h_kv": h_kv, "s_q": _log_int(rng, 256, 65536), "d": rng.choice([64, 128, 128]),
                "o": rng.choice(["f32", "f32", "bf16"]), "dtype": rng.choice(["bf16", "bf16", "f32"])}
    causal = rng.random() < 0.4
    s_q = _log_int(rng, 256, 32768 if kind == "bwd" else 49152)
    if rng.random() < 0.5:      # sequences are padded to tiles as often as not
        s_q = (s_q + 127) // 128 * 128
    s_k = s_q if causal or rng.random() < 0.7 else max(1, int(s_q * rng.uniform(0.5, 1.0)))
    case = {"kind": kind, "h_q": h_q, "h_kv": h_kv, "s_q": s_q, "s_k": s_k, "causal": causal}
    if kind == "fwd":
        case.update(acc=not causal and rng.random() < 0.6, o=rng.choice(["f32", "f32", "bf16"]))
    else:
        case.update(accumulate=rng.random() < 0.6)
    return case


def _d(case):
    return case.get("d", 128)


def _scale(case):
    return _d(case) ** -0.5


def _dtype(case):
    return DTYPES[case.get("dtype", "bf16")]


class _Rand:
    def __init__(self, seed):
        self.g = torch.Generator(device=DEV)
        self.g.manual_seed(seed)

    def __call__(self, *shape, dtype=torch.float32):
        if dtype == torch.float32 or math.prod(shape) < 1 << 28:
            return torch.randn(shape, generator=self.g, device=DEV).to(dtype)
        return torch.stack([torch.randn(shape[1:], generator=self.g, device=DEV).to(dtype) for _ in range(shape[0])])


def _lse_like(q, n_keys, scale):
    """The logsumexp that N(0, 1) keys give a query row, in expectation."""
    x = q.float()
    return math.log(n_keys) + 0.5 * scale * scale * (x * x).sum(-1)


def _partial(r, q, n_keys, scale, dtype=torch.float32):
    """An (o, lse) of the size that n_keys N(0, 1) keys and values give."""
    lse = _lse_like(q, n_keys, scale) + 0.05 * r(*q.shape[:2])
    return (r(*q.shape) * math.sqrt(math.e / n_keys)).to(dtype), lse


def _remote_workers(case):
    """Workers whose partials arrive at the last worker, in the order in which they are merged."""
    return [st.recv_from for st in dfa.dfa_schedule(case["p"], case["p"] - 1) if st.recv_from >= 0]


def _inputs(case, seed):
    """The tensors of a call, from the seed alone."""
    r, kind, d, dt, scale = _Rand(seed), case["kind"], _d(case), _dtype(case), _scale(case)
    h_q, h_kv = case["h_q"], case["h_kv"]
    x = {}
    if kind in ("schedule", "share", "autograd"):
        n, c = case["p"] * case["c"], case["c"]
        x["q"], x["do"] = r(h_q, n, d, dtype=dt), r(h_q, n, d, dtype=dt)
        x["k"], x["v"] = r(h_kv, n, d, dtype=dt), r(h_kv, n, d, dtype=dt)
        if kind == "share":
            x["remote"] = {h: _partial(r, x["q"][:, n - c:], c, scale) for h in _remote_workers(case)}
        return x
    s_q = case["s_q"]
    x["q"] = r(h_q, s_q, d, dtype=dt)
    if kind == "rows":
        odt = DTYPES[case["o"]]
        x["o_a"], x["lse_a"] = _partial(r, x["q"], s_q, scale, odt)
        x["o_b"], x["lse_b"] = _partial(r, x["q"], s_q, scale, odt)
        x["do"] = r(h_q, s_q, d, dtype=dt)
        return x
    x["k"], x["v"] = r(h_kv, case["s_k"], d, dtype=dt), r(h_kv, case["s_k"], d, dtype=dt)
    if kind == "fwd":
        if case["acc"]:
            x["o"], x["lse"] = _partial(r, x["q"], case["s_k"], scale, DTYPES[case["o"]])
        return x
    x["do"] = r(h_q, s_q, d, dtype=dt)
    # a diagonal chunk is taken as the sequence's first, an earlier one as one of four
    if case["causal"]:
        x["lse"] = _lse_like(x["q"], 1, scale) + torch.log(torch.arange(1, s_q + 1, device=DEV).float())
    else:
        x["lse"] = _lse_like(x["q"], 4 * case["s_k"], scale)
    x["delta"] = 0.1 * r(h_q, s_q)
    if case["accumulate"]:
        # sums of the size of this pair's own contributions
        held = case["s_k"] ** -0.5
        x["dq"], x["dk"], x["dv"] = held * r(h_q, s_q, d), held * r(h_kv, case["s_k"], d), held * r(h_kv, case["s_k"], d)
    return x


def prepare(case, seed):
    x, kind, d = _inputs(case, seed), case["kind"], _d(case)
    st = {"case": dict(case), "x": x}
    if kind in ("schedule", "share"):
        n = case["p"] * case["c"]
        st["bufs"] = driver.Buffers(case["h_q"], case["h_kv"], n, d, case["p"], DEV)
    elif kind == "autograd":
        for t in "qkv":
            x[t].requires_grad_(True)
        st["block"] = autograd.CheckpointedBlock(lambda o: o, _scale(case), case["p"], "attention_output")
    elif kind == "rows":
        x["delta"] = torch.empty(x["q"].shape[:2], device=DEV)
    elif kind == "fwd" and not case["acc"]:
        x["o"] = torch.empty(x["q"].shape, dtype=DTYPES[case["o"]], device=DEV)
        x["lse"] = torch.empty(x["q"].shape[:2], device=DEV)
    elif kind == "bwd" and not case["accumulate"]:
        x["dq"] = torch.empty(x["q"].shape, device=DEV)
        x["dk"], x["dv"] = torch.empty(x["k"].shape, device=DEV), torch.empty(x["k"].shape, device=DEV)
    return st


def run(st):
    case, x, kind, scale = st["case"], st["x"], st["case"]["kind"], _scale(st["case"])
    if kind == "schedule":
        b = st["bufs"]
        driver.run_all_workers(x["q"], x["k"], x["v"], x["do"], scale, case["p"], b)
        return {"o": b.O, "lse": b.L, "dq": b.dQ, "dk": b.dK, "dv": b.dV}
    if kind == "share":
        b, w, c = st["bufs"], case["p"] - 1, case["c"]
        driver.run_worker_share(x["q"], x["k"], x["v"], x["do"], scale, case["p"], w, b, x["remote"])
        lo = _first_chunk(case) * c
        return {"o": b.O[:, w * c:], "lse": b.L[:, w * c:], "dq": b.dQ[:, w * c:], "dk": b.dK[:, lo:], "dv": b.dV[:, lo:]}
    if kind == "autograd":
        q, k, v = x["q"], x["k"], x["v"]
        q.grad = k.grad = v.grad = None
        o = st["block"](q, k, v)
        o.backward(x["do"])
        return {"o": o.detach(), "dq": q.grad, "dk": k.grad, "dv": v.grad}
    if kind == "rows":
        dfa.dfa_merge(x["o_a"], x["lse_a"], x["o_b"], x["lse_b"])
        dfa.dfa_delta(x["o_a"], x["do"], delta=x["delta"])
        return {"o": x["o_a"], "lse": x["lse_a"], "delta": x["delta"]}
    if kind == "fwd":
        f = dfa.dfa_chunk_fwd_acc if case["acc"] else dfa.dfa_chunk_fwd
        o, lse = f(x["q"], x["k"], x["v"], case["causal"], scale, o=x["o"], lse=x["lse"])
        return {"o": o, "lse": lse}
    dfa.dfa_chunk_bwd(x["q"], x["k"], x["v"], x["lse"], x["delta"], x["do"], x["dq"], x["dk"], x["dv"], case["causal"],
                      scale, accumulate=case["accumulate"])
    return {"dq": x["dq"], "dk": x["dk"], "dv": x["dv"]}


def _first_chunk(case):
    """The earliest chunk whose keys the last worker attends to itself."""
    p = case["p"]
    return p - 1 - p // 2


def work(case):
    kind, d, h_q, h_kv = case["kind"], _d(case), case["h_q"], case["h_kv"]
    b = 2 if _dtype(case) == torch.bfloat16 else 4
    if kind == "rows":
        bo, rows = 2 if case["o"] == "bf16" else 4, h_q * case["s_q"]
        return {"bytes": rows * (3 * d * bo + 3 * 4 + d * b + 4), "flops": rows * d * 5}
    if kind in ("schedule", "share", "autograd"):
        c = case["c"]
        if kind == "share":
            own = case["p"] // 2
            nnz, s_q, s_k, partials = c * (c + 1) // 2 + own * c * c, c, (own + 1) * c, len(_remote_workers(case))
        else:
            n = case["p"] * c
            nnz, s_q, s_k, partials = n * (n + 1) // 2, n, n, 0
        grad = b if kind == "autograd" else 4
        out = h_q * s_q * d * (grad + (0 if kind == "autograd" else 4)) + 2 * h_kv * s_k * d * grad
        out += h_q * s_q * (d * b if kind == "autograd" else 4)
        moved = h_q * s_q * d * 2 * b + 2 * h_kv * s_k * d * b + out + partials * h_q * s_q * (d + 1) * 4
        return {"bytes": moved, "flops": 14 * d * h_q * nnz}
    s_q, s_k = case["s_q"], case["s_k"]
    nnz = s_q * (s_q + 1) // 2 if case["causal"] else s_q * s_k
    if kind == "fwd":
        bo = 2 if case["o"] == "bf16" else 4
        state = h_q * s_q * (d * bo + 4) * (2 if case["acc"] else 1)
        return {"bytes": h_q * s_q * d * b + 2 * h_kv * s_k * d * b + state, "flops": 4 * d * h_q * nnz}
    grads = (h_q * s_q + 2 * h_kv * s_k) * d * 4 * (2 if case["accumulate"] else 1)
    return {"bytes": 2 * h_q * s_q * d * b + 2 * h_kv * s_k * d * b + 8 * h_q * s_q + grads, "flops": 10 * d * h_q * nnz}


def tolerance(case):
    kind = case["kind"]
    if kind == "rows":
        return {"rel": 1e-2 if case["o"] == "bf16" else 1e-5}
    if kind == "schedule":
        return {"rel": 1e-5}
    # bf16 weights and score gradients: each output is measured 2e-3 to 3e-3 from its 64-bit value
    return {"rel": 1e-2}


# ---- the same in 64 bits -------------------------------------------------------------------------

_ROWS = 2048      # query rows taken at a time


def _pair_scores(q, k, scale, r0, offset):
    """Scaled scores of query rows r0.. against all keys; offset: position of the rows' first key
    (None: every key is visible)."""
    s = (q @ k.t()) * scale
    if offset is not None:
        i = torch.arange(r0, r0 + q.shape[0], device=q.device)[:, None] + offset
        s.masked_fill_(torch.arange(k.shape[0], device=q.device)[None, :] > i, -math.inf)
    return s


def _attention(q, k, v, scale, offset, state=None):
    """(o, lse) of one head; state: a list of further (o, lse) to combine with."""
    o, lse = torch.empty_like(q), torch.empty(q.shape[0], dtype=q.dtype, device=q.device)
    for r0 in range(0, q.shape[0], _ROWS):
        sl = slice(r0, r0 + _ROWS)
        s = _pair_scores(q[sl], k, scale, r0, offset)
        l = torch.logsumexp(s, 1)
        os, ls = [torch.exp(s - l[:, None]) @ v], [l]
        for po, pl in state or []:
            os.append(po[sl].double()); ls.append(pl[sl].double())
        lse[sl] = torch.logsumexp(torch.stack(ls), 0)
        o[sl] = sum(a * torch.exp(b - lse[sl])[:, None] for a, b in zip(os, ls))
    return o, lse


def _gradients(q, k, v, do, lse, delta, scale, offset, dq, dk, dv):
    """Adds one head's gradients to dq, dk, dv."""
    for r0 in range(0, q.shape[0], _ROWS):
        sl = slice(r0, r0 + _ROWS)
        p = torch.exp(_pair_scores(q[sl], k, scale, r0, offset) - lse[sl, None])
        ds = p * (do[sl] @ v.t() - delta[sl, None]) * scale
        dq[sl] += ds @ k
        dk += ds.t() @ q[sl]
        dv += p.t() @ do[sl]


def exact(case, seed):
    if work(case)["flops"] > 2.5e14:
        return None
    x, kind, scale, g = _inputs(case, seed), case["kind"], _scale(case), case["h_q"] // case["h_kv"]
    f64 = dict(dtype=torch.float64, device=DEV)
    if kind == "rows":
        la, lb = x["lse_a"].double(), x["lse_b"].double()
        lse = torch.logaddexp(la, lb)
        o = x["o_a"].double() * torch.exp(la - lse)[..., None] + x["o_b"].double() * torch.exp(lb - lse)[..., None]
        return {"o": o, "lse": lse, "delta": (o * x["do"].double()).sum(-1)}
    h_q, h_kv, d = case["h_q"], case["h_kv"], _d(case)
    if kind in ("fwd", "bwd"):
        offset = 0 if case["causal"] else None
        q_lo, k_lo, states = 0, 0, [[] for _ in range(h_q)]
        if kind == "fwd" and case["acc"]:
            states = [[(x["o"][h], x["lse"][h])] for h in range(h_q)]
    else:
        n, c = x["q"].shape[1], case["c"]
        q_lo = n - c if kind == "share" else 0
        k_lo = _first_chunk(case) * c if kind == "share" else 0
        offset = q_lo - k_lo
        states = [[(o[h], l[h]) for o, l in x["remote"].values()] if kind == "share" else [] for h in range(h_q)]
    s_q, s_k = x["q"].shape[1] - q_lo, x["k"].shape[1] - k_lo
    out = {}
    if kind != "bwd":
        out["o"], out["lse"] = torch.empty(h_q, s_q, d, **f64), torch.empty(h_q, s_q, **f64)
    if kind != "fwd":
        out["dq"], out["dk"], out["dv"] = (torch.zeros(h, s, d, **f64) for h, s in ((h_q, s_q), (h_kv, s_k), (h_kv, s_k)))
        if kind == "bwd" and case["accumulate"]:
            for t in ("dq", "dk", "dv"):
                out[t] += x[t]
    for h in range(h_q):
        q, k, v = x["q"][h, q_lo:].double(), x["k"][h // g, k_lo:].double(), x["v"][h // g, k_lo:].double()
        if kind != "bwd":
            out["o"][h], out["lse"][h] = _attention(q, k, v, scale, offset, states[h])
        if kind != "fwd":
            do = x["do"][h, q_lo:].double()
            if kind == "bwd":
                lse, delta = x["lse"][h].double(), x["delta"][h].double()
            else:
                lse, delta = out["lse"][h], (do * out["o"][h]).sum(-1)
            _gradients(q, k, v, do, lse, delta, scale, offset, out["dq"][h], out["dk"][h // g], out["dv"][h // g])
    if kind == "autograd":
        del out["lse"]
    return out
