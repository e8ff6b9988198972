"""The split-plane matrix-core kernels (fp32, and bf16 with d < 128) where their tiling can go wrong: lengths around
the 32-token tiles and 128-row chunks, slots taken several at a time, slots cut into segments, every head
size, packed documents, and values whose bf16 planes matter.

Tolerance, fp32: every product carries a relative error of 2^-24 at most (the plane products that are not formed) and
sums of n terms in fp32 a few times 2^-24 sqrt(n), both of either sign; n <= 2048 here, so 1e-6 of the norm is ten
times what comes out (1.2e-7), and a lost middle plane (2^-9) or low plane (2^-17 = 8e-6) fails.  bf16: outputs are
rounded to 8 bits, 2^-8 = 4e-3 of a value at most."""
import numpy as np
import pytest

from tests.util import host_inputs, rel_l2, to_device, to_host

pytestmark = pytest.mark.gpu
LIMIT = {"f32": 1e-6, "bf16": 4e-3}


@pytest.fixture(scope="module")
def oracle():
    import oracle as o
    return o


def _want(oracle, x, bounds, lam, H):
    """Definition in 64 bits, document by document."""
    parts = []
    for a, b in zip(bounds[:-1], bounds[1:]):
        t = {n: v[:, a:b].astype(np.float64) for n, v in x.items()}
        d = np.arange(b - a)[:, None] - np.arange(b - a)[None]
        w = np.tril(np.ones((b - a, b - a)))[None]
        if lam is not None:
            w = np.where(d >= 0, np.float64(lam)[:, None, None] ** np.maximum(d, 0), 0.0)
            w = np.tile(w, (x["Q"].shape[0] // H, 1, 1))
        s = (t["Q"] @ t["K"].transpose(0, 2, 1)) * w
        g = (t["dO"] @ t["V"].transpose(0, 2, 1)) * w
        parts.append((s @ t["V"], g @ t["K"], g.transpose(0, 2, 1) @ t["Q"], s.transpose(0, 2, 1) @ t["dO"]))
    return [np.concatenate(p, axis=1) for p in zip(*parts)]


def _run(oracle, dtype, B, H, N, d, C, L, cu=None, lam=None, seed=5):
    from paper_2502_07563_amd import binding as bd
    x = host_inputs(seed, B * H, N, d, dtype)
    p = bd.Problem(B, H, N, d, C, L, dtype, cu, decay=lam)
    t = {n: to_device(v, B, H, dtype) for n, v in x.items()}
    O, P = bd.forward(p, t["Q"], t["K"], t["V"])
    dQ, dK, dV, _ = bd.backward(p, t["Q"], t["K"], t["V"], t["dO"], P)
    want = _want(oracle, x, [0, N] if cu is None else list(cu), lam, H)
    for name, got, ref in zip(("O", "dQ", "dK", "dV"), (O, dQ, dK, dV), want):
        err = rel_l2(to_host(got), ref)
        assert err <= LIMIT[dtype], (name, dtype, B, H, N, d, C, L, err)


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16), ("bf16", 32), ("bf16", 64)])
@pytest.mark.parametrize("lam", [None, 0.97, 1e-3])
def test_tile_edges(oracle, dtype, d, lam):
    """Lengths on both sides of a tile (32), a stage (64) and a chunk (128); slots shorter than a chunk, taken
    several at a time or not; a slot cut into segments (few workgroups, L = 1024)."""
    f = None if lam is None else np.array([lam, 1.0], dtype=np.float32)
    for N, C, L in ((1, 1, 0), (31, 32, 0), (33, 64, 0), (129, 128, 0), (255, 64, 0), (300, 50, 0), (1100, 64, 1024)):
        _run(oracle, dtype, 1, 2, N, d, C, L, lam=f)


@pytest.mark.parametrize("dtype,d", [("f32", 32), ("f32", 128), ("bf16", 64)])
def test_packed_documents_and_merged_slots(oracle, dtype, d):
    lens = [64, 1, 127, 128, 129, 65, 300, 31]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    _run(oracle, dtype, 1, 2, int(cu[-1]), d, 64, 64, cu=cu)
    # enough groups that 64-token slots are taken two at a time
    _run(oracle, dtype, 16, 16, 200, d, 64, 64)
    cu = np.array([0, 70, 200, 391], dtype=np.int32)
    _run(oracle, dtype, 1, 256, 391, d, 32, 32, cu=cu, lam=np.full(256, 0.9, dtype=np.float32))


@pytest.mark.parametrize("slots", [1, 3, 100])
@pytest.mark.parametrize("dtype,d,lam", [("f32", 64, None), ("f32", 16, 0.9), ("bf16", 32, 0.97), ("bf16", 128, 0.2)])
def test_forced_walk_lengths(oracle, monkeypatch, dtype, d, lam, slots):
    """LASP2_WALK_SLOTS on these kernels: one slot per walk, walks whose chunks begin inside a slot, a whole document per
    walk.  (bf16, d = 128: states and scores of three planes, so the bound is that of the output's rounding too.)"""
    monkeypatch.setenv("LASP2_WALK_SLOTS", str(slots))
    f = None if lam is None else np.array([lam, 1.0], dtype=np.float32)
    _run(oracle, dtype, 2, 2, 500, d, 48, 48, lam=f)
    lens = [47, 300, 1, 97]
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    _run(oracle, dtype, 1, 2, int(cu[-1]), d, 32, 96, cu=cu, lam=f)

@pytest.mark.parametrize("lam", [None, 0.97])
@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 32), ("bf16", 64)])
def test_a_sequence_that_continues_another(dtype, d, lam):
    """P that is not zero where the sequence starts: what a program that holds a later part of a sequence has (the states of the
    parts before it are in its prefixes).  One slot and several, lengths that are walked whole and others: O and dQ have its share."""
    import torch
    from paper_2502_07563_amd import binding as bd
    G, f = 2, None if lam is None else np.array([lam, 1.0], dtype=np.float32)
    lams = torch.ones(G, device="cuda").double() if lam is None else torch.from_numpy(f).cuda().double()
    for N, L in ((200, 256), (1000, 1024), (300, 128), (500, 64), (700, 96), (2000, 512)):
        x = {n: to_device(v, 1, G, dtype) for n, v in host_inputs(31, G, N, d, dtype).items()}
        p = bd.Problem(1, G, N, d, L if L < 128 else 128, L, dtype, decay=f)
        own, T = bd.alloc_states(p), -(-N // L)
        bd.lasp2_chunk_states(p, x["K"], x["V"], own)
        bd.lasp2_state_prefix(p, own, own)
        X = torch.randn(G, d, d, generator=torch.Generator(device="cuda").manual_seed(N), device="cuda")
        age = lams[:, None] ** (L * torch.arange(T, device="cuda"))
        P = (own.double() + (age[:, :, None, None] * X.double()[:, None])[None]).float()
        O, dQ = torch.full_like(x["Q"], float("nan")), torch.full_like(x["Q"], float("nan"))
        dK, dV = torch.empty_like(x["K"]), torch.empty_like(x["V"])
        bd.lasp2_attn_fwd(p, x["Q"], x["K"], x["V"], P, O)
        bd.lasp2_attn_bwd(p, x["Q"], x["K"], x["V"], x["dO"], P, dQ, dK, dV, bd.alloc_workspace(p))
        Q, K, V, dO = (x[n][0].double() for n in ("Q", "K", "V", "dO"))
        i = torch.arange(N, device="cuda")
        w = (lams[:, None, None] ** (i[:, None] - i[None]).clamp(min=0)) * (i[:, None] >= i[None])
        from_X = (lams[:, None] ** (i + 1))[..., None]
        want = (w * (Q @ K.transpose(1, 2).contiguous())) @ V + from_X * (Q @ X.double())
        err = ((O[0].double() - want).norm() / want.norm()).item()
        assert err <= LIMIT[dtype], ("O", dtype, d, lam, N, L, err)
        if T > 1:      # (lasp2_attn_bwd does not read P where every sequence is a single slot)
            want = (w * (dO @ V.transpose(1, 2).contiguous())) @ K + from_X * (dO @ X.double().transpose(1, 2).contiguous())
            err = ((dQ[0].double() - want).norm() / want.norm()).item()
            assert err <= LIMIT[dtype], ("dQ", dtype, d, lam, N, L, err)


@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 32), ("f32", 128)])
def test_rows_that_the_mask_keeps_from_a_nan_stay_finite(dtype, d):
    """A NaN in V at token j reaches O at j and later, one in dO and Q the rows of dV and dK at j and before:
    not the other rows of the tile it lies in."""
    import torch
    from paper_2502_07563_amd import binding as bd
    N, j = 400, 177
    x = {n: to_device(v, 1, 2, dtype) for n, v in host_inputs(9, 2, N, d, dtype).items()}
    p = bd.Problem(1, 2, N, d, 128, 0, dtype)
    good, P = bd.forward(p, x["Q"], x["K"], x["V"])
    V = x["V"].clone()
    V[:, :, j, 3] = float("nan")
    O, _ = bd.forward(p, x["Q"], x["K"], V)
    assert torch.isfinite(O[:, :, :j]).all() and torch.isnan(O[:, :, j:, 3]).all()
    assert rel_l2(to_host(O[:, :, :j]), to_host(good[:, :, :j])) <= LIMIT[dtype]
    dO = x["dO"].clone()
    dO[:, :, j, 3] = float("inf")
    _, gk, gv, _ = bd.backward(p, x["Q"], x["K"], x["V"], x["dO"], P)
    _, dK, dV, _ = bd.backward(p, x["Q"], x["K"], x["V"], dO, P)
    assert torch.isfinite(dV[:, :, j + 1:]).all() and not torch.isfinite(dV[:, :, :j + 1, 3]).any()
    assert torch.isfinite(dK[:, :, j + 1:]).all()
    assert rel_l2(to_host(dV[:, :, j + 1:]), to_host(gv[:, :, j + 1:])) <= LIMIT[dtype]


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_values_of_every_exponent_are_split(d):
    """States of single rows, k^T v, with elements of one factor from 2^-126 to 2^126 and the other's so that the product is an
    ordinary number.  Three planes hold all bits of a value above 2^-109, and of a smaller one those above 2^-133: half of
    that lost, an error of 2^-134 / 2^e at most for values from 2^e on.  Products and sums: 2^-24 for the plane products that are
    not formed, 2^-24 twice for the sum of the small ones and of all."""
    import torch
    from paper_2502_07563_amd import binding as bd
    e = torch.arange(-126, 127)
    N, gen = len(e), torch.Generator().manual_seed(d)
    sign = lambda: torch.where(torch.rand(1, 2, N, d, generator=gen) < 0.5, -1.0, 1.0)
    a, b = ((1 + torch.rand(1, 2, N, d, generator=gen)) * sign() for _ in range(2))
    small = torch.ldexp(a, e[:, None])
    other = torch.ldexp(b, (-e).clamp(-20, 100)[:, None])
    limit = 3 * 2.0 ** -24 + 2.0 ** (-134.0 - e.double())
    p = bd.Problem(1, 2, N, d, 1, 1, "f32")
    M = bd.alloc_states(p)
    for K, V in ((small, other), (other, small)):
        bd.lasp2_chunk_states(p, K.cuda(), V.cuda(), M)
        want = K.double()[..., :, None] * V.double()[..., None, :]
        err = ((M.cpu().double() - want) / want).abs().amax((0, 1, 3, 4))
        bad = torch.nonzero(err > limit).flatten()
        assert not len(bad), [(int(e[i]), err[i].item(), limit[i].item()) for i in bad[:5]]


@pytest.mark.parametrize("d", [16, 32, 64, 128])
def test_weighted_rows_are_split_exactly(d):
    """With decay a row is multiplied by its weight and split into planes, which hold more bits than fp32: the state of one row of
    weight w < 1 is as close to w k^T v as that of a row of weight 1 to k^T v (the weight itself, the same for all elements, is fitted).
    A product that is rounded to fp32 before it is split adds about as much as the state's own rounding: 1.24 of the error."""
    import torch
    from paper_2502_07563_amd import binding as bd
    G = 64
    gen = torch.Generator(device="cuda").manual_seed(3)
    K, V = (torch.randn(1, G, 2, d, generator=gen, device="cuda") for _ in range(2))
    K[:, :, 1] = 0

    def error(lam):
        p = bd.Problem(1, G, 2, d, 2, 2, "f32", decay=np.full(G, lam, dtype=np.float32))
        M = bd.alloc_states(p)
        bd.lasp2_chunk_states(p, K, V, M)
        want = (K[0, :, 0, :, None].double() * V[0, :, 0, None].double()).flatten()
        w = (M.double().flatten() / want).mean()
        assert abs(w.item() / lam - 1) <= 1e-6
        return ((M.double().flatten() - w * want) / (w * want)).square().mean().sqrt().item()
    one = error(1.0)
    for lam in (0.6, 0.9, 0.99, 0.999):
        print(d, lam, error(lam) / one, flush=True)
        assert error(lam) <= 1.15 * one, (d, lam, error(lam), one)


def _positive_inputs(N, d, dtype, seed):
    import torch
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    gen = torch.Generator().manual_seed(seed)
    return {n: (2.0 ** -5 * (0.125 + 0.875 * torch.rand(N, d, generator=gen))).to(tdt) for n in ("Q", "K", "V", "dO")}


def _same_range(got, want, tol, what):
    """Element by element: infinities where |want| is past fp32's range, within tol of the value elsewhere."""
    import torch
    got, past = got.double().cpu(), want.abs() > torch.finfo(torch.float32).max
    assert torch.equal(got[past], torch.sign(want[past]) * float("inf")), what
    err = ((got - want).abs() / want.abs())[~past]
    assert bool((err <= tol).all()), (what, err.max().item())


@pytest.mark.parametrize("C,L,walk", [(128, 256, ""), (48, 48, "3")])
@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype,d,value", [(t, d, v) for t, d in (("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 64))
                                           for v in (float("inf"), -float("inf"), 3.4e38) if t == "f32" or v != 3.4e38])
def test_infinities_and_values_above_the_largest_bf16(monkeypatch, dtype, d, value, lam, C, L, walk):
    """One element of K or V is infinite or close to fp32's largest value: chunk states, carried states, outputs and
    gradients are what sums in fp32 give, in the chunk concerned, the ones after it and the slots after it (walked one by one,
    or three at a time).  Everything else is positive and below 2^-5, so no sum has terms of both signs or leaves the
    range by itself.  Bound per element: a sum of n positive terms of d-term scores, (n + d) 2^-24, and the decay's exponent,
    400 log2(1/0.9) 2^-24; bf16 results 2^-8, half of the last of 8 bits.  (The reference has 1e300 for an infinity: what
    comes out past fp32's range stands for one.)"""
    import torch
    from paper_2502_07563_amd import binding as bd
    monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
    N, j = 400, 130                                # second chunk of the first walk
    tol = (N + d + 100) * 2.0 ** -24 + (2.0 ** -8 if dtype == "bf16" else 0.0)
    w = torch.ones(N, N, dtype=torch.float64)
    if lam is not None:
        i = torch.arange(N)
        w = float(np.float32(lam)) ** (i[:, None] - i[None]).double()
    w = w.tril()
    for name, col in (("K", 3), ("V", 5)):
        x = _positive_inputs(N, d, dtype, d)
        x[name][j, col] = value
        ref = {n: v.double() for n, v in x.items()}
        if np.isinf(value):
            ref[name][j, col] = 1e300 if value > 0 else -1e300
        p = bd.Problem(1, 1, N, d, C, L, dtype, decay=None if lam is None else np.array([lam], dtype=np.float32))
        t = {n: v.cuda().view(1, 1, N, d) for n, v in x.items()}
        M = bd.alloc_states(p)
        bd.lasp2_chunk_states(p, t["K"], t["V"], M)
        O, P = bd.forward(p, t["Q"], t["K"], t["V"])
        dQ, dK, dV, _ = bd.backward(p, t["Q"], t["K"], t["V"], t["dO"], P)
        s, g = w * (ref["Q"] @ ref["K"].T), w * (ref["dO"] @ ref["V"].T)
        for slot, a in enumerate(range(0, N, L)):
            b = min(a + L, N)
            _same_range(M[0, 0, slot], (ref["K"][a:b] * w[b - 1, a:b, None]).T @ ref["V"][a:b], (N + 100) * 2.0 ** -24, ("M", name, slot))
        for what, a, b in (("O", O, s @ ref["V"]), ("dQ", dQ, g @ ref["K"]), ("dK", dK, g.T @ ref["Q"]), ("dV", dV, s.T @ ref["dO"])):
            _same_range(a[0, 0], b, tol, (what, name))


def _softmax64(Q, K, V, dO, bounds, causal, q0):
    """The definition in 64 bits: queries are the tokens q0 .. of N keys, attending inside their document."""
    n, N, d = Q.shape[1], K.shape[1], Q.shape[2]
    i, j = np.arange(q0, q0 + n), np.arange(N)
    doc = lambda t: np.searchsorted(bounds[1:], t, side="right")
    ok = (doc(i)[:, None] == doc(j)[None]) & ((j[None] <= i[:, None]) | (not causal))
    s = np.where(ok, (Q @ K.transpose(0, 2, 1)) / np.sqrt(d), -np.inf)
    m = s.max(axis=2, keepdims=True)
    e = np.exp(s - m)
    lse = np.log(e.sum(axis=2)) + m[..., 0]
    p = e / e.sum(axis=2, keepdims=True)
    O = p @ V
    ds = p * (dO @ V.transpose(0, 2, 1) - (dO * O).sum(axis=2, keepdims=True)) / np.sqrt(d)
    return O, lse, ds @ K, ds.transpose(0, 2, 1) @ Q, p.transpose(0, 2, 1) @ dO


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 32), ("f32", 64), ("f32", 128), ("bf16", 16), ("bf16", 32), ("bf16", 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_softmax_tile_edges(dtype, d, causal):
    """Row counts around a tile (32), a stage (64, 128) and an odd number of mirrored tiles; a share of the
    queries; documents; enough groups for workgroups of four row tiles.  fp32: a probability carries the rounding
    of its exponent, 2^-24 |score| with scores below 8 here, and a gradient the difference of two such terms."""
    import torch
    from paper_2502_07563_amd import binding as bd
    limit = {"f32": 3e-6, "bf16": 6e-3}[dtype]
    cu3 = np.array([0, 33, 34, 300], dtype=np.int32)
    for G, N, q0, n, cu in ((2, 1, 0, 1, None), (2, 33, 0, 33, None), (3, 96, 0, 96, None), (2, 161, 0, 161, None), (2, 290, 193, 97, None),
                            (2, 300, 0, 300, cu3), (2, 300, 30, 100, cu3), (256, 150, 0, 150, None),
                            (520, 70, 0, 70, np.array([0, 37, 70], dtype=np.int32))):
        x = host_inputs(G + N, G, N, d, dtype)
        x = {k: v * np.float32(2.0) for k, v in x.items()}
        p = bd.Problem(1, G, N, d, 64, 0, dtype, cu)
        t = {k: to_device(v, 1, G, dtype) for k, v in x.items()}
        Q, dO = t["Q"][:, :, q0:q0 + n].contiguous(), t["dO"][:, :, q0:q0 + n].contiguous()
        nan = lambda like: torch.full_like(like, float("nan"))
        O, lse, dQ, dK, dV = nan(Q), torch.full((1, G, n), float("nan"), device="cuda"), nan(Q), nan(t["K"]), nan(t["V"])
        ws = torch.empty(bd.lasp2_softmax_share_workspace_size(p, n), dtype=torch.uint8, device="cuda")
        bd.lasp2_softmax_fwd_share(p, q0, n, Q, t["K"], t["V"], O, lse, causal)
        bd.lasp2_softmax_bwd_share(p, q0, n, Q, t["K"], t["V"], O, dO, lse, dQ, dK, dV, ws, causal)
        x64 = {k: v.astype(np.float64) for k, v in x.items()}
        bounds = np.array([0, N]) if cu is None else cu
        want = _softmax64(x64["Q"][:, q0:q0 + n], x64["K"], x64["V"], x64["dO"][:, q0:q0 + n], bounds, causal, q0)
        got = (to_host(O), lse.cpu().numpy()[0].astype(np.float64), to_host(dQ), to_host(dK), to_host(dV))
        # A row with a single key has dQ = dK = 0, the difference of two sums dO.v that are rounded apart: up to
        # 2^-23 |dO| |v| |k| / sqrt(d), with |v| |k| / sqrt(d) = 4 / sqrt(d) <= 1 here; 1.5e-7 of |dV| = |dO| is allowed.
        scale = np.linalg.norm(want[4])
        for name, a, b in zip(("O", "LSE", "dQ", "dK", "dV"), got, want):
            err = np.linalg.norm(a - b) / max(np.linalg.norm(b), 0.05 * scale)
            assert err <= limit, (name, dtype, d, causal, G, N, q0, n, err)


def _softmax_all(dtype, d, x, causal, cu=None):
    """O, LSE, dQ, dK, dV as 64-bit host tensors [N, d] ([N])."""
    import torch
    from paper_2502_07563_amd import binding as bd
    N = x["Q"].shape[0]
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    p = bd.Problem(1, 1, N, d, 64, 0, dtype, cu)
    Q, K, V, dO = (x[n].to(tdt).cuda().view(1, 1, N, d) for n in ("Q", "K", "V", "dO"))
    O, dQ, dK, dV = (torch.empty_like(Q) for _ in range(4))
    lse = torch.empty(1, 1, N, device="cuda")
    ws = torch.empty(bd.lasp2_softmax_workspace_size(p), dtype=torch.uint8, device="cuda")
    bd.lasp2_softmax_fwd(p, Q, K, V, O, lse, causal)
    bd.lasp2_softmax_bwd(p, Q, K, V, O, dO, lse, dQ, dK, dV, ws, causal)
    return [t[0, 0].double().cpu() for t in (O, lse, dQ, dK, dV)]


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 64)])
def test_softmax_rows_that_the_mask_keeps_from_a_nan_stay_finite(dtype, d):
    """A NaN in V at token j reaches O at j and later in the same document, one in dO (and so in its delta) at token i the
    rows of dV and dK at i and before: not the other rows of the tile, nor the next document in it."""
    import torch
    N, cu = 300, np.array([0, 90, 300], dtype=np.int32)
    x = {n: 2 * torch.randn(N, d, generator=torch.Generator().manual_seed(ord(n[-1]))) for n in ("Q", "K", "V", "dO")}
    good = _softmax_all(dtype, d, x, True, cu)
    limit = {"f32": 1e-5, "bf16": 1e-2}[dtype]     # (four and two times the error of a row allowed above)
    j = 77                                         # documents meet at 90: both lie in the tile 64 .. 95
    y = dict(x, V=x["V"].clone())
    y["V"][j, 3] = float("nan")
    O, lse, dQ = _softmax_all(dtype, d, y, True, cu)[:3]
    free = (torch.arange(N) < j) | (torch.arange(N) >= 90)
    assert torch.isnan(O[~free, 3]).all() and torch.isfinite(O[~free][:, [2, 4]]).all()
    assert torch.isfinite(lse).all() and torch.isfinite(O[free]).all() and torch.isfinite(dQ[free]).all()
    assert rel_l2(O[free], good[0][free]) <= limit and rel_l2(dQ[free], good[2][free]) <= limit
    y = dict(x, dO=x["dO"].clone())
    y["dO"][95, 3] = float("nan")                  # sixth token of the second document
    dQ, dK, dV = _softmax_all(dtype, d, y, True, cu)[2:]
    free = (torch.arange(N) < 90) | (torch.arange(N) > 95)
    assert torch.isnan(dV[~free, 3]).all() and torch.isnan(dK[~free]).all() and torch.isnan(dQ[95]).all()
    assert torch.isfinite(dV[free]).all() and torch.isfinite(dK[free]).all() and torch.isfinite(dQ[torch.arange(N) != 95]).all()
    assert rel_l2(dV[free], good[4][free]) <= limit and rel_l2(dK[free], good[3][free]) <= limit


@pytest.mark.parametrize("dtype,d", [("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 64)])
@pytest.mark.parametrize("causal", [True, False])
def test_softmax_infinite_keys_and_large_values(dtype, d, causal):
    """Queries are positive, so a key with an element of -inf has scores of -inf and probability 0: the layer is that
    without the key, with dK = dV = 0 for it.  fp32: a value of 3.4e38, above
    the largest bf16, is taken as the finite number that it is."""
    import torch
    N, j = 300, 70
    limit = {"f32": 1e-5, "bf16": 1e-2}[dtype]
    x = {n: torch.randn(N, d, generator=torch.Generator().manual_seed(ord(n[-1]))) for n in ("Q", "K", "V", "dO")}
    x["Q"] = x["Q"].abs() + 0.1
    x["K"][j, 3] = -float("inf")
    O, lse, dQ, dK, dV = _softmax_all(dtype, d, x, causal)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    r = {n: v.to(tdt).double() for n, v in x.items()}
    r["K"][j, 3] = -1e9                            # exp of it is 0 in 64 bits too
    n64 = {n: v.numpy()[None] for n, v in r.items()}
    want = [torch.from_numpy(t[0]) for t in _softmax64(n64["Q"], n64["K"], n64["V"], n64["dO"], np.array([0, N]), causal, 0)]
    for what, a, b in (("O", O, want[0]), ("LSE", lse[:, None], want[1][:, None]), ("dV", dV, want[4])):
        assert rel_l2(a, b) <= limit, what
    # dS = 0 for the key: 0 * inf in dQ's column 3 for the rows that see it, as in any arithmetic; dK has no such term
    assert torch.equal(dK[j], torch.zeros(d, dtype=torch.float64)) and torch.equal(dV[j], torch.zeros(d, dtype=torch.float64))
    cols = [c for c in range(d) if c != 3]
    assert rel_l2(dQ[:, cols], want[2][:, cols]) <= limit and rel_l2(dK, want[3]) <= limit
    if dtype == "f32":
        x["K"][j, 3] = 0.0
        x["V"][j, 5] = 3.4e38
        O = _softmax_all(dtype, d, x, causal)[0]
        n64 = {n: v.double().numpy()[None] for n, v in x.items()}
        p = _softmax64(n64["Q"], n64["K"], n64["V"], n64["dO"], np.array([0, N]), causal, 0)[0][0]
        assert torch.isfinite(O).all()
        assert rel_l2(O[:, 5], p[:, 5]) <= limit
        cols = [c for c in range(d) if c != 5]
        assert rel_l2(O[:, cols], p[:, cols]) <= limit
