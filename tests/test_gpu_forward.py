"""lasp2_forward: O and every entry of P against the definition in 64 bits and against the three calls it stands for.
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
    (128, 0, 1, [700]), (64, 0, 0, [100, 4000]), (256, 0, 0, [1531]),
]


@pytest.mark.gpu
@pytest.mark.parametrize("decay", [False, True])
@pytest.mark.parametrize("C,L,walk,docs", CASES)
def test_forward_in_one_call(monkeypatch, C, L, walk, docs, decay):
    if walk:
        monkeypatch.setenv("LASP2_WALK_SLOTS", str(walk))
    cu = np.concatenate([[0], np.cumsum(docs)]).astype(np.int32)
    H, N, d = 3, int(cu[-1]), 128
    B = 2 if len(docs) == 1 else 1
    lam = np.array([1 - 2.0 ** -5, 0.9, 1.0], np.float32) if decay else None
    p = bd.Problem(B, H, N, d, C, L, "bf16", cu if len(docs) > 1 else None, decay=lam)
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
    # fp32 sums over at most 4000 tokens; with decay every token's weighted row is rounded to bf16 (2^-9 of it)
    tol = 2.0 ** -8 if decay else 4000 * 2.0 ** -24
    for got in (P, P3):
        err = (got.double() - want).norm(dim=(3, 4))
        assert bool((err <= tol * size).all()), (err / size).max().item()
    diff = (O.float() - O3.float()).norm(dim=3)
    # the same products; states that differ in rounding order only: a rounding of O, the scores and the snapshot each
    assert bool((diff <= 3 * 2.0 ** -8 * O3.float().norm(dim=3) + 1e-6).all())
