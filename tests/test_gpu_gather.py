"""Linear attention, bf16 heads of 128: walks that gather the state they start from, with as many rows before (and, in the backward,
behind) them as fill the ring of stages partly, exactly and several times, with ragged last stages and sums of 512 rows on both
sides; and tensors that fill the last cache, whose rows are then loaded past it.  Against the definition in 64 bits."""
import numpy as np
import pytest
import torch

from paper_2502_07563_amd import binding as bd


def _problem(G, N, L, lam=None, device="cuda"):
    f = None if lam is None else np.full(G, lam, np.float32)
    return bd.Problem(1, G, N, 128, 64, L, "bf16", decay=f, device=device)


def _want(x, lam):
    q, k, v, w = (t.double() for t in x)
    i = torch.arange(q.shape[0], device="cuda")
    m = torch.tril(lam ** (i[:, None] - i[None]).clamp(min=0).double())
    s, g = m * (q @ k.T.contiguous()), m * (w @ v.T.contiguous())
    return s @ v, g @ k, g.T.contiguous() @ q, s.T.contiguous() @ w


def _check(G, N, L, lam, heads, rows):
    p = _problem(G, N, L, lam)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = [torch.randn(1, G, N, 128, generator=gen, device="cuda").mul_(128 ** -0.5).to(torch.bfloat16) for _ in range(4)]
    O, P = bd.forward(p, *x[:3])
    alone = torch.empty_like(O)
    bd.lasp2_attn_fwd(p, *x[:3], P, alone)
    got = (O,) + bd.backward(p, *x, P)[:3]
    for s in range(0, N, L):   # sums of at most N rows in fp32; with decay a row is rounded to bf16 when it has been weighted
        w = (1.0 if lam is None else lam) ** torch.arange(s - 1, -1, -1, device="cuda").double()[:, None]
        for h in heads:
            want = (x[1][0, h, :s].double() * w).T.contiguous() @ x[2][0, h, :s].double()
            err = (P[0, h, s // L].double() - want).norm().item()
            assert err <= (4096 * 2.0 ** -24 if lam is None else 2.0 ** -8) * want.norm().item(), ("P", G, N, L, lam, h, s, err)
    for h in heads:
        want = _want([t[0, h] for t in x], 1.0 if lam is None else lam)
        for name, a, b in list(zip(("O", "dQ", "dK", "dV"), got, want)) + [("attn_fwd", alone, want[0])]:
            a = a[0, h].double()
            # results, scores, the state's snapshot and, with decay, the weighted rows are rounded to bf16 (2^-9 each at most,
            # half of that in the mean); every 64 rows on their own, so that a wrong block does not drown in the others
            for r in range(0, N, rows):
                err = ((a[r:r + rows] - b[r:r + rows]).norm() / b[r:r + rows].norm()).item()
                assert err <= 2.0 ** -7, (name, G, N, L, lam, h, r, err)


# rows of the sequence; walks of 128 or 256 gather 0, 64 .. 2 560 rows from its start and to its end
LENGTHS = (129, 191, 320, 321, 383, 449, 512, 575, 769, 1024, 1025, 1087, 1531, 2111, 2700)


def test_the_lengths_gather():
    """(256 CUs assumed where no device answers)"""
    for N in LENGTHS[2:]:
        assert bd.lasp2_walk_plan(_problem(2, N, 4096, device="cpu"), "forward") == (128, "gather"), N
    assert any(bd.lasp2_walk_plan(_problem(2, N, 4096, device="cpu"), "attn_bwd")[1] == "gather" for N in LENGTHS)


@pytest.mark.gpu
@pytest.mark.parametrize("lam", [None, 0.99])
@pytest.mark.parametrize("N", LENGTHS)
def test_rows_gathered(N, lam):
    for L in (64, 128, 256, 4096):
        _check(2, N, L, lam, (0, 1), 64)


@pytest.mark.gpu
@pytest.mark.parametrize("G,N,L", [(2, 1500, 128), (4, 1531, 128), (16, 1024, 256)])
def test_heads_that_do_not_decay_are_summed_as_without_decay(G, N, L):
    """Factors of 1 beside others.  Weights are 1, rows are exact, and P is off by what sums in fp32 round: of 512 rows and then of
    those sums without decay, of 128 and then of those with it, in walks that add a slot's rows to all of the state before
    them.  Counting roundings, each of the sum so far: not more than without decay, whose walks round the states inside them
    alike (one sum of all rows: 1.4 times; measured 0.8, and 1.4)."""
    lam = np.where(np.arange(G) % 2 == 0, 1.0, 1.0 - 2.0 ** -12).astype(np.float32)
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = [torch.randn(1, G, N, 128, generator=gen, device="cuda").mul_(128 ** -0.5).to(torch.bfloat16) for _ in range(3)]
    want = torch.stack([x[1][0, ::2, :s].double().transpose(1, 2).contiguous() @ x[2][0, ::2, :s].double() for s in range(0, N, L)], 1)
    err = []
    for decay in (None, lam):
        p = bd.Problem(1, G, N, 128, 64, L, "bf16", decay=decay)
        assert bd.lasp2_walk_plan(p, "forward")[1] == "gather"
        P = bd.forward(p, *x)[1]
        err.append(((P[0, ::2].double() - want).norm() / want.norm()).item())
    print(G, N, L, err, err[1] / err[0], flush=True)
    assert err[1] <= 1.25 * err[0], (G, N, L, err)


BOTH_SIDES = [(16, 2048, 128, 128), (17, 1930, 128, 256), (24, 1400, 128, 256), (32, 1024, 512, 128), (33, 1024, 512, 256), (40, 385, 4096, 128),
              # walks end with their slots: 11 and 16 of a sequence's walks, not 8 and 12; 192 and 256 tokens are a slot, most of one
              (16, 1000, 192, 128), (16, 1536, 192, 128), (16, 1600, 192, 192), (32, 1000, 192, 192), (16, 1600, 320, 128), (16, 2048, 320, 256)]


def test_the_sides_of_256_workgroups():
    """(256 CUs assumed where no device answers)"""
    for G, N, L, rows in BOTH_SIDES:
        assert bd.lasp2_walk_plan(_problem(G, N, L, device="cpu"), "forward") == (rows, "gather"), (G, N, L)


@pytest.mark.gpu
@pytest.mark.parametrize("G,N,L", [c[:3] for c in BOTH_SIDES] + [(16, 2049, 128), (256, 129, 256)])
def test_walks_of_128_rows_and_of_256(G, N, L):
    """Both sides of 256 workgroups of 128 rows, and of the first choice, walks that gather."""
    _check(G, N, L, None, (0, G - 1), 64)


@pytest.mark.gpu
@pytest.mark.parametrize("G,N,L,lam", [(128, 4096, 512, None), (2048, 250, 256, None), (128, 4096, 512, 0.99), (16, 32768, 4096, None)])
def test_tensors_that_fill_the_cache(G, N, L, lam):
    """Two tensors of 128 MiB.  (Long sequences: the first walks' rows only, by the rows that follow them.)"""
    if N <= 4096:
        _check(G, N, L, lam, (0, 77, G - 1), 64)
        return
    p, n = _problem(G, N, L, lam), 4096 + 300
    gen = torch.Generator(device="cuda").manual_seed(N)
    x = [torch.randn(1, G, N, 128, generator=gen, device="cuda").mul_(128 ** -0.5).to(torch.bfloat16) for _ in range(4)]
    O, P = bd.forward(p, *x[:3])
    dQ = bd.backward(p, *x, P)[0]
    for h in (0, G - 1):
        want = _want([t[0, h, :n] for t in x], 1.0)
        for name, a, b in (("O", O, want[0]), ("dQ", dQ, want[1])):
            err = ((a[0, h, :n].double() - b).norm() / b.norm()).item()
            assert err <= 2.0 ** -7, (name, h, err)
