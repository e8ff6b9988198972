"""What the library's users have it do, as timed cases: attention layers, forward and backward.

`listed()` names the workloads that this repository's configurations, tests and benchmark use, from the
smallest call to the long-sequence training step; `draw()` gives more of the same ranges.  Every
pass goes through the public entry points of `paper_2502_07563_amd.binding`.

Fields of a case
  op      "linear" (LASP-2 with masking), "nomask" (without), "softmax" (standard attention of the hybrid model)
  dtype, B, H, N, d, C, L   the descriptor (L = 0: one state per chunk)
  docs    0, or the number of documents packed into the N tokens (lengths lognormal, at least 64 tokens)
  decay   linear: per-head factors 1 - 2^(-5-h)
  train   forward and backward; otherwise the forward alone (prefill)
  serial  linear: one slot per sequence, no state arrays (P = None)
  causal, q_len   softmax: the mask, and the number of queries: the last q_len tokens of the N (0: all of them)
"""
import math

import numpy as np
import torch

from paper_2502_07563_amd import binding as bd
from paper_2502_07563_amd import synth


def _case(name=None, op="linear", dtype="bf16", B=1, H=16, N=1024, d=128, C=256, L=0, docs=0, decay=False,
          train=True, serial=False, causal=True, q_len=0):
    c = dict(op=op, dtype=dtype, B=B, H=H, N=N, d=d, C=C, L=L, docs=docs, decay=decay, train=train,
             serial=serial, causal=causal, q_len=q_len)
    if name:
        c["name"] = name
    return c


def listed():
    return [
        # the small fp32 layer that numerics are checked with (configuration 1): a few short launches
        _case("fp32_d64_1k", dtype="f32", H=2, N=1024, d=64, C=128),
        # prefill of one prompt of ordinary, odd length: forward alone, far too small to fill the device
        _case("prefill_1531", N=1531, train=False),
        # training step, 1B model's layer, 32K tokens, one state per chunk (configuration 2)
        _case("train_32k", N=32768),
        # the headline: one 256K-token sequence, slots of 4096 tokens (configuration 3)
        _case("train_256k", N=262144, L=4096),
        # training step, 8B model's layer, a batch of 8K sequences (configuration 4)
        _case("train_batch_8k", B=8, H=32, N=8192),
        # packed variable-length batch: 40 documents in 131072 tokens (configuration 5)
        _case("train_packed", H=32, N=131072, docs=40),
        # scalar decay (Retention / Lightning Attention form), 128K tokens
        _case("train_decay_128k", N=131072, L=4096, decay=True),
        # bidirectional layer, without masking, odd length
        _case("nomask_100k", op="nomask", N=100003, L=4096),
        # standard-attention layer of the hybrid model, whole sequence, causal
        _case("softmax_32k", op="softmax", N=32768, C=64),
        # the same layer, one rank's share: the last 4096 queries against 131072 gathered keys
        _case("softmax_share_128k", op="softmax", N=131072, C=64, q_len=4096),
        # linear layer with heads of 64, bf16, odd length
        _case("bf16_d64_4k", B=4, H=16, N=4001, d=64, C=128),
        # fp32 standard attention of a small model, odd length
        _case("softmax_fp32_2k", op="softmax", dtype="f32", H=8, N=2003, d=64, C=64),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case.  Lengths are spread over their logarithm and mostly not multiples of a tile; the number of
    rows (or of query-key pairs) is capped at that of the listed case of the same kind."""
    kind = rng.choice(["linear"] * 5 + ["decay", "nomask", "softmax", "softmax", "plain", "plain", "plain_softmax"])
    H = rng.choice([4, 8, 12, 16, 20, 32])
    B = rng.choice([1, 1, 1, 2, 4, 8])
    C = rng.choice([64, 128, 256, 256])
    train = rng.random() < 0.75
    if kind in ("linear", "decay", "nomask"):
        most = {"linear": 16 * 262144, "decay": 16 * 131072, "nomask": 16 * 100003}[kind]
        N = _log_int(rng, 200, min(262144, most // (B * H)))
        L = rng.choice([0, 0, 1024, 2048, 4096])
        docs = 0
        if B == 1 and N >= 4096 and rng.random() < 0.4:
            docs = min(rng.randint(3, 60), N // 256)
        serial = kind == "linear" and not docs and B * H >= 64 and rng.random() < 0.3
        if serial:
            L = -(-N // C) * C
        return _case(op="nomask" if kind == "nomask" else "linear", B=B, H=H, N=N, C=C, L=L, docs=docs,
                     decay=kind == "decay", train=train, serial=serial)
    if kind == "softmax":
        pairs = 16 * 32768 * 32768 // 2
        causal = rng.random() < 0.7
        share = rng.random() < 0.3
        N = _log_int(rng, 200, int(math.sqrt(pairs / (B * H) * (2 if causal else 1))))
        docs = min(rng.randint(3, 40), N // 256) if B == 1 and not share and N >= 2048 and rng.random() < 0.4 else 0
        return _case(op="softmax", B=B, H=H, N=N, C=64, docs=docs, train=train, causal=causal,
                     q_len=max(1, N // rng.choice([4, 8, 16])) if share else 0)
    dtype, d = rng.choice([("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 64)])
    if kind == "plain":
        N = _log_int(rng, 200, min(16384, 4 * 16 * 4001 * 64 // (d * B * H)))
        return _case(dtype=dtype, B=B, H=H, N=N, d=d, C=min(C, 128), L=rng.choice([0, 0, 512, 1024]),
                     decay=rng.random() < 0.3, train=train)
    B, H = 1, min(H, 16)
    N = _log_int(rng, 100, int(math.sqrt(8 * 2003 * 2003 * 64 / (d * H))))
    return _case(op="softmax", dtype=dtype, B=B, H=H, N=N, d=d, C=64, train=train, causal=rng.random() < 0.7)


def _offsets(c):
    """Document offsets of a packed case (a property of the case, like its sizes)."""
    return synth.doc_offsets(4, c["N"], c["docs"], c["N"] / c["docs"], 64) if c["docs"] else None


def _q_len(c):
    return c["q_len"] or c["N"]


def prepare(case, seed):
    """Inputs of one layer in device memory, the descriptor, and for softmax the buffers a program keeps.
    Linear layers: normal / sqrt(d), as the benchmark draws them; softmax layers: unit variance."""
    c = case
    gen = torch.Generator(device="cuda")
    gen.manual_seed(seed)
    tdt = torch.bfloat16 if c["dtype"] == "bf16" else torch.float32
    scale = 1.0 if c["op"] == "softmax" else 1.0 / math.sqrt(c["d"])

    def mk(n):
        return torch.randn((c["B"], c["H"], n, c["d"]), generator=gen, device="cuda").mul_(scale).to(tdt)
    decay = (1.0 - 2.0 ** (-5.0 - np.arange(c["H"]))).astype(np.float32) if c["decay"] else None
    p = bd.Problem(c["B"], c["H"], c["N"], c["d"], c["C"], c["L"], c["dtype"], _offsets(c), decay=decay)
    s = {"c": c, "p": p, "Q": mk(_q_len(c)), "K": mk(c["N"]), "V": mk(c["N"])}
    if c["train"]:
        s["dO"] = mk(_q_len(c))
    if c["op"] == "softmax":
        s["O"] = torch.empty_like(s["Q"])
        s["LSE"] = torch.empty(s["Q"].shape[:3], dtype=torch.float32, device="cuda")
        if c["train"]:
            s["dQ"], s["dK"], s["dV"] = torch.empty_like(s["Q"]), torch.empty_like(s["K"]), torch.empty_like(s["V"])
            s["ws"] = torch.empty(bd.lasp2_softmax_share_workspace_size(p, _q_len(c)), dtype=torch.uint8, device="cuda")
    elif c["serial"]:
        s["O"] = torch.empty_like(s["Q"])
        if c["train"]:
            s["dQ"], s["dK"], s["dV"] = (torch.empty_like(s["Q"]) for _ in range(3))
            s["ws"] = bd.alloc_workspace(p)
    return s


def run(state):
    """One pass: the layer's forward and, when training, its backward."""
    s, c, p = state, state["c"], state["p"]
    Q, K, V = s["Q"], s["K"], s["V"]
    if c["op"] == "softmax":
        if c["q_len"]:
            q0, n = c["N"] - c["q_len"], c["q_len"]
            bd.lasp2_softmax_fwd_share(p, q0, n, Q, K, V, s["O"], s["LSE"], c["causal"])
            if not c["train"]:
                return s["O"], s["LSE"]
            bd.lasp2_softmax_bwd_share(p, q0, n, Q, K, V, s["O"], s["dO"], s["LSE"], s["dQ"], s["dK"], s["dV"],
                                       s["ws"], c["causal"])
        else:
            bd.lasp2_softmax_fwd(p, Q, K, V, s["O"], s["LSE"], c["causal"])
            if not c["train"]:
                return s["O"], s["LSE"]
            bd.lasp2_softmax_bwd(p, Q, K, V, s["O"], s["dO"], s["LSE"], s["dQ"], s["dK"], s["dV"], s["ws"],
                                 c["causal"])
        return s["O"], s["LSE"], s["dQ"], s["dK"], s["dV"]
    if c["op"] == "nomask":
        O, S = bd.nomask_forward(p, Q, K, V)
        if not c["train"]:
            return O, S
        return (O, S) + bd.nomask_backward(p, Q, K, V, s["dO"], S)[:3]
    if c["serial"]:
        bd.lasp2_attn_fwd(p, Q, K, V, None, s["O"])
        if not c["train"]:
            return s["O"]
        bd.lasp2_attn_bwd(p, Q, K, V, s["dO"], None, s["dQ"], s["dK"], s["dV"], s["ws"])
        return s["O"], s["dQ"], s["dK"], s["dV"]
    O, P = bd.forward(p, Q, K, V)
    if not c["train"]:
        return O, P
    return (O, P) + bd.backward(p, Q, K, V, s["dO"], P)[:3]


def _slots(c):
    L = c["L"] or c["C"]
    cu = _offsets(c)
    lens = [c["N"]] if cu is None else [int(b - a) for a, b in zip(cu[:-1], cu[1:])]
    return sum(-(-n // L) for n in lens)


def _pairs(c):
    """(query, key) pairs inside the mask, per head."""
    n = _q_len(c)
    if c["docs"]:
        lens = [float(x) for x in np.diff(_offsets(c))]
        return sum(x * (x + 1) / 2 if c["causal"] else x * x for x in lens)
    return n * (c["N"] - n) + n * (n + 1) / 2.0 if c["causal"] else float(n) * c["N"]


def work(case):
    """Each input read once and each output written once (state arrays that the caller gets included).
    Operations: linear layers, the state products alone (2 per token forward, 4 backward, of 2 d^2 each), which is
    what the recurrence needs however the tokens are tiled; softmax, 2 products per pair forward and 5 backward."""
    c = case
    e = 2 if c["dtype"] == "bf16" else 4
    G, d, n, N = c["B"] * c["H"], c["d"], _q_len(c), c["N"]
    tens = G * d * e
    if c["op"] == "softmax":
        b = tens * (2 * n + 2 * N) + 4 * G * n                  # Q, O, K, V, LSE
        f = 4.0 * G * _pairs(c) * d
        if c["train"]:
            b += tens * (2 * n + 2 * N)                         # dO, dQ, dK, dV
            f += 10.0 * G * _pairs(c) * d
        return {"bytes": float(b), "flops": f}
    b = tens * N * (8 if c["train"] else 4) + (0 if c["serial"] else 4 * G * _slots(c) * d * d)
    return {"bytes": float(b), "flops": float(G * N * d * d * (12 if c["train"] else 4))}


def tolerance(case):
    # About four times the difference from the same path in 64 bits, measured on outputs and gradients at lengths of
    # 1000 to 4000 tokens: bf16 2.3e-3 .. 2.9e-3 with d = 128 (scores and state operands are rounded to bf16) and
    # 1.6e-3 .. 1.8e-3 with d = 64 (outputs alone); fp32 2.3e-7 .. 3e-7 in linear layers, 4e-7 .. 1.1e-6 in softmax.
    if case["dtype"] == "bf16":
        return {"rel": 1e-2 if case["d"] == 128 else 7e-3}
    return {"rel": 5e-6 if case["op"] == "softmax" else 1.5e-6}


def _chunked64(Q, K, V, dO, lam, C, L):
    """Causal linear attention of one document in 64 bits, [G,n,d] tensors: O, the states before each slot of L
    tokens, dQ, dK, dV (chunks of C tokens, one state carried from chunk to chunk).  lam: [G] factors, or None."""
    G, n, d = Q.shape
    T = -(-n // C)
    a = torch.arange(C, device=Q.device, dtype=torch.float64)
    lam = torch.ones(G, dtype=torch.float64, device=Q.device) if lam is None else lam
    pw = lam[:, None] ** torch.arange(C + 1, device=Q.device)                       # [G,C+1]
    W = torch.tril(lam[:, None, None] ** (a[:, None] - a[None, :]).clamp(min=0))[:, None]
    up = lambda x: None if x is None else torch.nn.functional.pad(x, (0, 0, 0, T * C - n)).view(G, T, C, d)
    Q, K, V, dO = up(Q), up(K), up(V), up(dO)
    tr = lambda x: x.transpose(-1, -2).contiguous()
    down = lambda x: x.reshape(G, T * C, d)[:, :n]

    def carry(M, order):
        out, S = torch.empty_like(M), torch.zeros_like(M[:, 0])
        for t in order:
            out[:, t] = S
            S = pw[:, C, None, None] * S + M[:, t]
        return out
    S = carry(tr(K * pw[:, :C].flip(1)[:, None, :, None]) @ V, range(T))
    grow = pw[:, 1:][:, None, :, None]
    O = down((W * (Q @ tr(K))) @ V + grow * (Q @ S))
    P = S[:, ::L // C]
    if dO is None:
        return O, P
    R = carry(tr(Q * pw[:, :C][:, None, :, None]) @ dO, range(T - 1, -1, -1))
    fall = pw[:, 1:].flip(1)[:, None, :, None]
    dQ = down((W * (dO @ tr(V))) @ K + grow * (dO @ tr(S)))
    del S
    dK = down((tr(W) * (V @ tr(dO))) @ Q + fall * (V @ tr(R)))
    return O, P, dQ, dK, down((tr(W) * (K @ tr(Q))) @ dO + fall * (K @ R))


def _softmax64(Q, K, V, dO, causal, q0):
    """Softmax attention of one document in 64 bits, [n,d] queries at positions q0.. against [N,d] keys:
    O, log-sum-exp, dQ, dK, dV, in blocks of 2048 queries."""
    (n, d), N = Q.shape, K.shape[0]
    O, lse = torch.empty_like(Q), Q.new_empty(n)
    dQ, dK, dV = (torch.zeros_like(x) for x in (Q, K, V))
    for i in range(0, n, 2048):
        j = min(n, i + 2048)
        m = q0 + j if causal else N
        s = (Q[i:j] @ K[:m].T).div_(math.sqrt(d))
        if causal:
            at = torch.arange(q0 + i, q0 + j, device=Q.device)
            s.masked_fill_(torch.arange(m, device=Q.device)[None] > at[:, None], -math.inf)
        lse[i:j] = torch.logsumexp(s, 1)
        p = s.sub_(lse[i:j, None]).exp_()
        O[i:j] = p @ V[:m]
        if dO is not None:
            g = dO[i:j]
            dV[:m] += p.T @ g
            ds = (g @ V[:m].T).sub_((g * O[i:j]).sum(1, keepdim=True)).mul_(p).div_(math.sqrt(d))
            dQ[i:j] = ds @ K[:m]
            dK[:m] += ds.T @ Q[i:j]
    return (O, lse) if dO is None else (O, lse, dQ, dK, dV)


def exact(case, seed):
    """What run() returns, from the definitions in 64 bits with torch alone."""
    c = case
    s = prepare(c, seed)
    B, H, G, N = c["B"], c["H"], c["B"] * c["H"], c["N"]
    Q, K, V, dO = (s[n].double().view(G, -1, c["d"]) if n in s else None for n in ("Q", "K", "V", "dO"))
    cu = [0, N] if not c["docs"] else [int(x) for x in _offsets(c)]
    part = lambda x, g, lo, hi: None if x is None else x[g, lo:hi]
    if c["op"] == "softmax":
        heads = []
        for g in range(G):
            docs = []
            for lo, hi in zip(cu[:-1], cu[1:]):
                ql, qh = (0, c["q_len"]) if c["q_len"] else (lo, hi)
                docs.append(_softmax64(Q[g, ql:qh], K[g, lo:hi], V[g, lo:hi], part(dO, g, ql, qh), c["causal"],
                                       N - c["q_len"] if c["q_len"] else 0))
            heads.append([torch.cat(x) for x in zip(*docs)])
        return tuple(torch.stack(x).view((B, H) + x[0].shape) for x in zip(*heads))
    if c["op"] == "nomask":
        tr = lambda x: x.transpose(-1, -2).contiguous()
        L, outs = c["L"] or c["C"], []
        for lo, hi in zip(cu[:-1], cu[1:]):
            q, k, v, g = (part(x, slice(None), lo, hi) for x in (Q, K, V, dO))
            S = tr(k) @ v
            out = [q @ S, S[:, None].expand(-1, -(-(hi - lo) // L), -1, -1)]
            if g is not None:
                R = tr(q) @ g
                out += [g @ tr(S), v @ tr(R), k @ R]
            outs.append(out)
    else:
        lam = None
        if c["decay"]:
            lam = torch.from_numpy((1.0 - 2.0 ** (-5.0 - np.arange(H))).astype(np.float32)).cuda().double().repeat(B)
        outs = [_chunked64(*(part(x, slice(None), lo, hi) for x in (Q, K, V, dO)), lam, c["C"], c["L"] or c["C"])
                for lo, hi in zip(cu[:-1], cu[1:])]
    out = [torch.cat(x, 1) for x in zip(*outs)]
    if c["serial"]:
        del out[1]
    out = [x.reshape((B, H) + x.shape[1:]) for x in out]
    return out[0] if len(out) == 1 else tuple(out)
