"""lasp2_forward: O and every entry of P against the definition in 64 bits and against the three calls it stands for; and
the gradients.  Short sequences are one launch each way, whose walks gather the states they start from (the first
cases); one head or two of a long one gets its states from the states kernel (the last cases).
Walks of several slots write the states inside them in passing: slot lengths of one and of an odd number of 64-token
blocks, walks whose last slot, last block or last row is the sequence's, documents of one walk and of several."""
import numpy as np
import pytest
import torch

from paper_2502_07563_amd import binding as bd

CASES = [  # C, L, walk slots (0: the library's choice), lengths of the documents
    (64, 0, 4, [1500]), (64, 0, 3, [64 * 9 + 1]), (64, 0, 5, [64 * 10]), (64, 0, 8, [449]), (192, 0, 2, [1000]),
    (128, 0, 2, [1025]), (128, 0, 16, [1931]), (256, 0, 2, [1536]), (256, 512, 2, [2047]), (64, 320, 3, [2000]),
    (64, 0, 4, [1, 64, 65, 700, 256, 257, 320]), (256, 0, 4, [3000, 5, 1024, 1025]), (100, 0, 3, [1000]),
    (128, 0, 1, [700]), (64, 0, 0, [100, 4000]), (256, 0, 0, [1531]), (256, 0, 0, [63]), (64, 0, 0, [257]),
    (64, 0, 0, [9001]), (256, 0, 0, [16384]), (128, 384, 5, [12000]), (64, 0, 7, [9999]), (64, 0, 0, [13000, 1, 129, 64]),
    # long slots, cut into walks: one slot, several, a last slot shorter than a walk, documents
    (256, 7168, 0, [7000]), (256, 4096, 0, [8200]), (256, 4096, 0, [9000]), (128, 1920, 0, [7700]), (100, 1000, 0, [3500]),
    (256, 2048, 0, [5000, 70, 2049]), (64, 4096, 0, [4096, 257, 4200, 5]),
    # walks of single slots: of 128 rows and fewer, of between 128 and 256, and forced
    (128, 0, 0, [300]), (100, 0, 0, [245]), (192, 0, 0, [380]), (256, 0, 1, [500]),
]


def _case(monkeypatch, C, L, walk, docs, decay, device="cuda"):
    if walk:
        monkeypatch.setenv("LASP2_WALK_SLOTS", str(walk))
    else:
        monkeypatch.delenv("LASP2_WALK_SLOTS", raising=False)
    cu = np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)
    N, d = int(cu[-1]), 128
    B, H = (2 if len(docs) == 1 else 1, 3) if N < 5000 else (1, 2)
    lam = np.array([1 - 2.0 ** -5, 0.9, 1.0], np.float32)[:H] if decay else None
    return bd.Problem(B, H, N, d, C, L, "bf16", cu if len(docs) > 1 else None, decay=lam, device=device), cu, lam


@pytest.mark.parametrize("decay", [False, True])
def test_the_cases_take_every_route(monkeypatch, decay):
    """What the library chooses for the cases below (256 CUs assumed where no device answers): each call's walks of several slots,
    of one and of parts of one, for each kind of start that it has."""
    routes = set()
    for C, L, walk, docs in CASES:
        p, cu, _ = _case(monkeypatch, C, L, walk, docs, decay, "cpu")
        for call in bd.CALLS:
            w, start = bd.lasp2_walk_plan(p, call)
            lone = max(docs) <= (w if start == "states" else L or C)
            routes.add((call, start, "part" if w < (L or C) else "one" if w == (L or C) else "several", lone))
    states = {("states", kind, lone) for kind in ("one", "several") for lone in (False, True)}
    alone = {("states", kind, True) for kind in ("one", "several")}
    gather = {("gather", "one", False), ("gather", "several", False), ("gather", "part", False)}
    want = {(call,) + r for call in bd.CALLS for r in states | {("gather", "part", True), ("slots", "part", False)}}
    want |= {(call,) + r for call in ("forward", "attn_bwd") for r in gather}
    if not decay:   # (whole documents without decay: few of them gather, many are for the full sizes)
        want -= {("attn_bwd",) + r for r in alone}
        want.add(("attn_bwd", "gather", "one", True))
    assert want <= routes, sorted(want - routes)


@pytest.mark.gpu
@pytest.mark.parametrize("decay", [False, True])
@pytest.mark.parametrize("C,L,walk,docs", CASES)
def test_forward_in_one_call(monkeypatch, C, L, walk, docs, decay):
    p, cu, lam = _case(monkeypatch, C, L, walk, docs, decay)
    B, H, N, d = p.B, p.H, p.N, p.d
    gen = torch.Generator(device="cuda").manual_seed(N + C)
    Q, K, V = (torch.randn(B, H, N, d, generator=gen, device="cuda").mul_(d ** -0.5).to(torch.bfloat16) for _ in range(3))
    P, O = bd.alloc_states(p).fill_(float("nan")), torch.full_like(Q, float("nan"))
    bd.lasp2_forward(p, Q, K, V, P, O)
    P3, O3 = bd.alloc_states(p), torch.empty_like(Q)
    bd.lasp2_chunk_states(p, K, V, P3)
    bd.lasp2_state_prefix(p, P3, P3)
    bd.lasp2_attn_fwd(p, Q, K, V, P3, O3)

    want, at, Ls = torch.zeros(P.shape, dtype=torch.float64, device="cuda"), 0, L or C
    lamt = torch.ones(H, dtype=torch.float64) if lam is None else torch.from_numpy(lam.astype(np.float64))
    for a, b in zip(cu[:-1], cu[1:]):
        for s in range(a, b, Ls):
            if s > a:
                w = lamt[:, None].cuda() ** torch.arange(s - 1 - a, -1, -1, device="cuda")
                k = (K[:, :, a:s].double() * w[None, :, :, None]).transpose(2, 3).contiguous()
                want[:, :, at] = k @ V[:, :, a:s].double()
            at += 1
    assert at == P.shape[2]
    size = want.norm(dim=(3, 4)).clamp_min(1e-30)
    # fp32 sums over at most N tokens; with decay every token's weighted row is rounded to bf16 (2^-9 of it)
    tol = 2.0 ** -8 if decay else max(N, 4000) * 2.0 ** -24
    for got in (P, P3):
        err = (got.double() - want).norm(dim=(3, 4))
        assert bool((err <= tol * size).all()), (err / size).max().item()
    diff = (O.float() - O3.float()).norm(dim=3)
    # the same products; states that differ in rounding order only: a rounding of O, the scores and the snapshot each
    assert bool((diff <= 3 * 2.0 ** -8 * O3.float().norm(dim=3) + 1e-6).all())

    dO = torch.randn(B, H, N, d, generator=gen, device="cuda").mul_(d ** -0.5).to(torch.bfloat16)
    grads = bd.backward(p, Q, K, V, dO, P)[:3]
    tr = lambda x: x.transpose(-1, -2).contiguous()
    for a, b in zip(cu[:-1], cu[1:]):
        for g in range(B * H):
            q, k, v, w = (x.reshape(B * H, N, d)[g, a:b].double() for x in (Q, K, V, dO))
            i = torch.arange(b - a, device="cuda")
            m = torch.tril(lamt[g % H].item() ** (i[:, None] - i[None, :]).clamp(min=0).double())
            s, t = m * (q @ tr(k)), m * (w @ tr(v))
            # what a result's terms add up to in quadrature if every score has the size of its own terms: a lone row whose
            # score happens to be small keeps the rounding of the products it is the sum of
            size = lambda x, y: (m * (x.norm(dim=1)[:, None] * y.norm(dim=1)[None, :]) / d ** 0.5) ** 2
            ss, ts = size(q, k), size(w, v)
            refs = (("O", O, s @ v, ss @ v ** 2), ("dQ", grads[0], t @ k, ts @ k ** 2),
                    ("dK", grads[1], tr(t) @ q, tr(ts) @ q ** 2), ("dV", grads[2], tr(s) @ w, tr(ss) @ w ** 2))
            for name, got, ref, terms in refs:
                diff = (got.reshape(B * H, N, d)[g, a:b].double() - ref)
                # operands, scores, snapshot and result each rounded to bf16: per 64 rows at most their sum, 2^-9 each
                for r in range(0, b - a, 64):
                    err, by = diff[r:r + 64].norm().item(), terms[r:r + 64].sum().sqrt().item()
                    assert err <= 5 * 2.0 ** -9 * by, (name, g, a + r, err / by)

    if P.shape[2] == len(docs):   # every document one slot: no states are needed
        none = [torch.full_like(Q, float("nan")) for _ in range(4)]
        bd.lasp2_attn_fwd(p, Q, K, V, None, none[0])
        bd.lasp2_attn_bwd(p, Q, K, V, dO, None, *none[1:], bd.alloc_workspace(p))
        assert torch.equal(none[0], O3) and all(torch.equal(x, y) for x, y in zip(none[1:], grads))


@pytest.mark.gpu
@pytest.mark.parametrize("C,walk,N", [(64, 0, 707), (64, 8, 3050), (256, 2, 3050), (64, 3, 1000)])
def test_decayed_states_of_walks_weigh_rows_within_64(monkeypatch, C, walk, N):
    """States at a walk's start with a factor so close to one that weights round to it in bf16: a row's weight
    counts within its 64 rows only, so it is off by 63 * (1 - factor) at most however long the walk is."""
    if walk:
        monkeypatch.setenv("LASP2_WALK_SLOTS", str(walk))
    H, d, near = 3, 128, 2.0 ** -16
    lam = np.full(H, 1.0 - near, dtype=np.float32)
    gen = torch.Generator(device="cuda")
    gen.manual_seed(N)
    Q, K, V = (torch.randn(1, H, N, d, generator=gen, device="cuda").mul_(d ** -0.5).to(torch.bfloat16) for _ in range(3))
    P = bd.forward(bd.Problem(1, H, N, d, C, 0, "bf16", decay=lam), Q, K, V)[1]
    i = torch.arange(N, device="cuda", dtype=torch.float64)
    for t in range(1, P.shape[2]):
        a = t * C
        w = float(lam[0]) ** (a - 1 - i[:a])
        ref = torch.bmm((K[0, :, :a].double() * w[None, :, None]).transpose(1, 2).contiguous(), V[0, :, :a].double())
        # 2^-14: 64 roundings in fp32 of sums and factors.  (A slot of C rows that no walk starts in counts within 64 rows too.)
        assert (P[0, :, t].double() - ref).norm() <= (63 * near + 2.0 ** -14) * ref.norm(), t
