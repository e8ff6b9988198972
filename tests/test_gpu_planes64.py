"""Linear attention with heads of 64 (fp32, bf16): walks of several slots that write the states of the slots inside them, against
the definition in 64 bits: lengths on both sides of a chunk of 64 rows and of a tile of 32, slots of whole chunks (the states are
written in passing) and others (they are not), one slot per walk, several, whole documents, segments of a walk, documents, decay;
infinities, whose chunks are done again in fp32 and whose states have to come out there too."""
import numpy as np
import pytest
import torch

from paper_2502_07563_amd import binding as bd
from tests.test_gpu_planes import LIMIT

pytestmark = pytest.mark.gpu


def _inputs(G, N, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    return [(torch.randn(1, G, N, 64, generator=gen, device="cuda") / 8).to(tdt) for _ in range(4)]


def _want(x, cu, L, lam):
    """O, P, dQ, dK, dV in 64 bits; lam: [G]"""
    out = []
    for a, b in zip(cu[:-1], cu[1:]):
        Q, K, V, dO = (t[0, :, a:b].double() for t in x)
        i = torch.arange(b - a, device="cuda")
        w = (lam[:, None, None] ** (i[:, None] - i[None]).clamp(min=0)) * (i[:, None] >= i[None])
        s, g = w * (Q @ K.transpose(1, 2).contiguous()), w * (dO @ V.transpose(1, 2).contiguous())
        P = [torch.zeros_like(K[:, :64, :64].new_zeros(K.shape[0], 64, 64))]
        for j in range(L, b - a, L):
            P.append((K[:, :j] * (lam[:, None] ** (j - 1 - i[None, :j]))[..., None]).transpose(1, 2).contiguous() @ V[:, :j])
        out.append((s @ V, torch.stack(P, 1), g @ K, g.transpose(1, 2).contiguous() @ Q, s.transpose(1, 2).contiguous() @ dO))
    return [torch.cat(t, 1) for t in zip(*out)]


def _check(dtype, G, N, L, docs=None, lam=None, seed=3):
    cu = np.concatenate([[0], np.cumsum(docs or [N])]).astype(np.int32)
    x = _inputs(G, N, dtype, seed)
    f = None if lam is None else np.linspace(lam, 1.0, G).astype(np.float32)
    p = bd.Problem(1, G, N, 64, L if L < 64 else 64 if L % 64 == 0 else L, L, dtype, cu if docs else None, decay=f)
    lams = torch.ones(G, dtype=torch.float64, device="cuda") if f is None else torch.from_numpy(f).cuda().double()
    want = _want(x, cu, L, lams)
    O, P = bd.forward(p, *x[:3])
    got = (O, P) + bd.backward(p, *x, P)[:3]
    alone = torch.full_like(O, float("nan"))
    bd.lasp2_attn_fwd(p, *x[:3], P, alone)
    for name, a, b in list(zip(("O", "P", "dQ", "dK", "dV"), got, want)) + [("attn_fwd", alone, want[0])]:
        err = ((a[0].double() - b).norm() / max(b.norm().item(), 1e-30)).item()
        assert err <= (LIMIT["f32"] if name == "P" else LIMIT[dtype]), (name, dtype, G, N, L, docs, lam, err)


@pytest.mark.parametrize("walk", ["", "1", "2", "3", "100"])
@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_walks(monkeypatch, dtype, lam, walk):
    monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
    for N, L in ((1, 64), (32, 64), (33, 64), (63, 64), (65, 64), (128, 64), (191, 64), (449, 64), (700, 128), (513, 192), (300, 50), (900, 512)):
        _check(dtype, 2, N, L, lam=lam)
    for L in (64, 128, 96):
        _check(dtype, 3, 64 + 1 + 200 + 129 + 63, L, docs=[64, 1, 200, 129, 63], lam=lam)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_many_groups(dtype):
    """Both sides of the choice: whole sequences in one launch, walks of several slots, a launch per kind; two or one
    workgroups per CU, segments of one chunk and of more."""
    for G, N, L in ((16, 1000, 64), (48, 512, 64), (48, 513, 64), (48, 768, 64), (48, 769, 64), (130, 300, 128), (60, 1030, 64), (16, 2000, 512), (130, 1025, 64)):
        _check(dtype, G, N, L)


@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_states_of_slots_behind_an_infinity(monkeypatch, dtype, lam, value):
    """An element of K that is not finite, in the first, a middle and the last row of a chunk: the states that the walks write are
    finite, infinite or NaN where those of states and prefix kernels are (one slot per walk), and so are the outputs."""
    N, L = 500, 64
    f = None if lam is None else np.array([lam, 1.0], dtype=np.float32)
    p = bd.Problem(1, 2, N, 64, 64, L, dtype, decay=f)
    for j in (0, 130, 191, 499):
        Q, K, V, _ = _inputs(2, N, dtype, j)
        K[0, 1, j, 3] = value
        got = []
        for walk in ("1", "3", "100"):
            monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
            got.append(bd.forward(p, Q, K, V))
        for O, P in got[1:]:
            for a, b in ((O, got[0][0]), (P, got[0][1])):
                assert torch.equal(torch.isfinite(a), torch.isfinite(b)), j
                assert torch.equal(torch.isnan(a), torch.isnan(b)), j
                ok = torch.isfinite(b)
                assert ((a[ok].double() - b[ok].double()).norm() / b[ok].double().norm()).item() <= 4 * LIMIT[dtype], j
        assert torch.isfinite(got[1][1][0, 0]).all()


def _suffix(x, cu, L, lam):
    """What follows each slot of its document, Q^T dO in 64 bits as the slot's end sees it; lam: [G]"""
    out = []
    for a, b in zip(cu[:-1], cu[1:]):
        Q, dO = x[0][0, :, a:b].double(), x[3][0, :, a:b].double()
        for end in range(L, b - a + L, L):
            i = torch.arange(max(b - a - end, 0), device="cuda")
            out.append((Q[:, end:] * (lam[:, None] ** i)[..., None]).transpose(1, 2).contiguous() @ dO[:, end:])
    return torch.stack(out, 1)


@pytest.mark.parametrize("walk", ["", "1", "3", "100"])
@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype,d", [("f32", 64), ("bf16", 64), ("f32", 16), ("bf16", 32), ("f32", 128)])
def test_the_workspace_holds_the_suffix_of_every_slot(monkeypatch, dtype, d, lam, walk):
    """lasp2_attn_bwd on the split-plane kernels, whatever its walks are: slots that the walks write in passing and others, whole
    sequences in one walk, segments of a walk, documents.  (Sums of at most 4 001 products in fp32: as P in _check.)"""
    monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
    docs = [64, 1, 200, 129, 63, 500]
    for G, N, L, lens in ((2, 65, 64, None), (2, 191, 64, None), (16, 1000, 64, None), (4, 500, 128, None), (2, 4001, 128, None), (64, 900, 128, None),
                          (2, 700, 192, None), (3, 300, 50, None), (40, 640, 64, None), (2, 900, 512, None),
                          (3, sum(docs), 64, docs), (3, sum(docs), 128, docs), (3, sum(docs), 96, docs)):
        cu = np.concatenate([[0], np.cumsum(lens or [N])]).astype(np.int32)
        x = [t[..., :d].contiguous() if d <= 64 else torch.cat([t, t.flip(-1)], -1) for t in _inputs(G, N, dtype, N)]
        f = None if lam is None else np.linspace(lam, 1.0, G).astype(np.float32)
        p = bd.Problem(1, G, N, d, L if L < 64 else 64 if L % 64 == 0 else L, L, dtype, cu if lens else None, decay=f)
        lams = torch.ones(G, dtype=torch.float64, device="cuda") if f is None else torch.from_numpy(f).cuda().double()
        P, ws = bd.forward(p, *x[:3])[1], bd.alloc_workspace(p).fill_(float("nan"))
        grads = [torch.empty_like(t) for t in x[:3]]
        bd.lasp2_attn_bwd(p, *x, P, *grads, ws)
        want = _suffix(x, cu, L, lams)
        got = bd.workspace_states(p, ws)[0].double()
        err = ((got - want).norm() / want.norm()).item()
        assert err <= LIMIT["f32"], (dtype, d, lam, walk, G, N, L, lens, err)
        for a, b in zip((-1,) if lens is None else np.cumsum([-(-n // L) for n in lens]) - 1, (-1,) if lens is None else range(len(lens))):
            assert not got[:, a].any(), (dtype, d, lam, walk, G, N, L, lens, b)   # nothing follows a document's last slot


@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("value", [float("inf"), float("nan")])
def test_suffixes_of_slots_before_an_infinity(monkeypatch, dtype, lam, value):
    """The same for an element of dO that is not finite and the suffixes that the backward's walks write."""
    N, L = 500, 64
    f = None if lam is None else np.array([lam, 1.0], dtype=np.float32)
    p = bd.Problem(1, 2, N, 64, 64, L, dtype, decay=f)
    for j in (0, 130, 191, 499):
        Q, K, V, dO = _inputs(2, N, dtype, j)
        P = bd.forward(p, Q, K, V)[1]
        dO[0, 1, j, 3] = value
        got = []
        for walk in ("1", "3", "100"):
            monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
            got.append(bd.backward(p, Q, K, V, dO, P))
        for other in got[1:]:
            for a, b in zip(other, got[0]):
                assert torch.equal(torch.isfinite(a), torch.isfinite(b)), j
                assert torch.equal(torch.isnan(a), torch.isnan(b)), j
                ok = torch.isfinite(b)
                assert ((a[ok].double() - b[ok].double()).norm() / b[ok].double().norm()).item() <= 4 * LIMIT[dtype], j
        assert torch.isfinite(got[1][3][0, 0]).all()


@pytest.mark.parametrize("lam", [None, 0.9])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_walks_of_several_slots_are_as_accurate_as_slots(monkeypatch, dtype, lam):
    """States are sums of slots' sums however many slots a walk has.  Error of P and of the suffixes against 64 bits, walks of
    several slots against slots one by one.  A sum of n rows, 16 at a time, rounds n / 16 times something that grows to the
    result: slots of 64 and then their sums n / 64 times, so that one running sum would be off by up to twice as much
    (1.2 to 1.9 measured at these sizes); the same sums in another order differ by a few per cent, heads with factors of
    their own taken together (the rounding of a factor is the same in all of a head's slots)."""
    for G, N, L in ((16, 1000, 64), (16, 4001, 64), (32, 2001, 128), (64, 4001, 128)):
        x = _inputs(G, N, dtype, 17)
        f = np.ones(G, dtype=np.float32) if lam is None else np.linspace(lam, 1.0, G).astype(np.float32)
        p = bd.Problem(1, G, N, 64, 64, L, dtype, decay=None if lam is None else f)
        lams = torch.from_numpy(f).cuda().double()
        # (prefixes are the suffixes of the rows in reverse, those of a whole number of slots)
        cut = (N - 1) // L * L
        back = [None if t is None else t[:, :, :cut].flip(2) for t in (x[1], None, None, x[2])]
        want = _suffix(back, [0, cut], L, lams).flip(1), _suffix(x, [0, N], L, lams)
        err = {}
        for walk in ("1", ""):
            monkeypatch.setenv("LASP2_WALK_SLOTS", walk)
            P = bd.forward(p, *x[:3])[1]
            S = bd.backward(p, *x, P)[3]
            err[walk] = [((a[0, :, :b.shape[1]].double() - b).norm() / b.norm()).item() for a, b in zip((P, S), want)]
        for name, one, several in zip(("P", "suffix"), err["1"], err[""]):
            print(name, dtype, lam, G, N, L, one, several, flush=True)
            assert several <= 1.1 * one, (name, dtype, lam, G, N, L, one, several)
