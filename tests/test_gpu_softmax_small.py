"""bf16 heads of 128, softmax: the kernels for launches of at most a workgroup of 64 rows per CU and those for more (the
same lengths with many heads), against the definition in 64 bits: one row more or less than row tiles, steps of 128 partner
rows and blocks of 256 queries; mirrored row tiles with an odd number of them; documents; one rank's share, with fewer
queries than a tile and with forward and dK, dV on different sides of a line; few partner rows, which the kernels for more take."""
import numpy as np
import pytest
import torch

from paper_2502_07563_amd import binding as bd

SIZES = [(1, None, None), (31, None, None), (65, None, None), (95, None, None), (128, None, None), (129, None, None), (257, None, None),
         (321, None, None), (700, None, None), (420, None, (32, 63, 33, 65, 64, 163)), (600, (500, 100), None), (600, (37, 5), None),
         (500, (499, 1), None), (512, (128, 300), (100, 412)), (300, (300, 0), None),
         # beside the numbers of partner rows from which the kernels for small launches are taken
         (160, None, None), (161, None, None), (192, None, None), (193, None, None), (193, None, (60, 70, 63)), (400, (150, 43), None)]


@pytest.mark.gpu
@pytest.mark.parametrize("causal", [False, True])
@pytest.mark.parametrize("per_cu", [0, 64, 128])   # two heads, or just too many for that many rows per workgroup and CU
@pytest.mark.parametrize("N,share,docs", SIZES)
def test_bf16_d128(N, share, docs, per_cu, causal):
    q0, n = share or (0, N)
    cus = torch.cuda.get_device_properties(0).multi_processor_count
    H = cus // -(-max(n, 1) // per_cu) + 1 if per_cu else 2
    d, cu = 128, np.concatenate([[0], np.cumsum(docs or [N])]).astype(np.int32)
    p = bd.Problem(1, H, N, d, 64, 0, "bf16", cu if docs else None)
    gen = torch.Generator(device="cuda").manual_seed(N + n)
    mk = lambda k: torch.randn(1, H, k, d, generator=gen, device="cuda").to(torch.bfloat16)
    Q, K, V, dO = mk(n), mk(N), mk(N), mk(n)
    nan = lambda x: torch.full_like(x, float("nan"))
    O, dQ, dK, dV = nan(Q), nan(Q), nan(K), nan(V)
    lse = torch.full((1, H, n), float("nan"), device="cuda")
    ws = torch.full((max(bd.lasp2_softmax_share_workspace_size(p, n) // 4, 4),), float("nan"), device="cuda")
    bd.lasp2_softmax_fwd_share(p, q0, n, Q, K, V, O, lse, causal)
    bd.lasp2_softmax_bwd_share(p, q0, n, Q, K, V, O, dO, lse, dQ, dK, dV, ws, causal)
    for g in {0, H // 2, H - 1}:
        q, k, v, w, o = (x[0, g].double() for x in (Q, K, V, dO, O))
        i, j = torch.arange(q0, q0 + n, device="cuda")[:, None], torch.arange(N, device="cuda")[None]
        doc = torch.from_numpy(np.repeat(np.arange(len(cu) - 1), np.diff(cu))).cuda()
        keep = doc[q0:q0 + n, None] == doc[None]
        if causal:
            keep &= j <= i
        s = (q @ k.T / d ** 0.5).masked_fill(~keep, -float("inf"))
        P = torch.softmax(s, 1) if n else s
        if n:
            assert (lse[0, g].double() - torch.logsumexp(s, 1)).abs().max().item() <= 1e-4
        # Per row, against the row with the terms of each sum in quadrature: 2^-9 each for the rounded probabilities (or dS), for
        # what enters through O's own rounding, and for the result; scores are fp32.
        dp, dl = w @ v.T, (w * o).sum(1, keepdim=True)
        ds, size = P * (dp - dl) / d ** 0.5, P * (dp.abs() + dl.abs()) / d ** 0.5
        for name, got, want, terms in (("O", O, P @ v, P ** 2 @ v ** 2), ("dQ", dQ, ds @ k, size ** 2 @ k ** 2),
                                       ("dK", dK, ds.T @ q, (size ** 2).T @ q ** 2), ("dV", dV, P.T @ w, (P ** 2).T @ w ** 2)):
            err = (got[0, g].double() - want).norm(dim=1)
            assert bool((err <= 4 * 2.0 ** -9 * torch.maximum(terms.sum(1).sqrt(), want.norm(dim=1)) + 1e-30).all()), (name, g)
