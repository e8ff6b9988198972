"""The small passes between the large kernels, against 64-bit sums.  Prefix and suffix of the states: where the
walk's batches of eight slots and the documents' borders meet (fewer slots than a batch, one more or less,
several documents in a batch).  Row sums of the softmax backward: every head size and type, numbers of
rows beside those of a workgroup."""
import numpy as np
import pytest
import torch

from paper_2502_07563_amd import binding as bd

C = 16


@pytest.mark.gpu
@pytest.mark.parametrize("in_place", [False, True])
@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("decay", [False, True])
@pytest.mark.parametrize("d,slots", [(16, [1]), (64, [7]), (128, [8]), (32, [9]), (128, [16]), (64, [17]), (128, [33]),
                                     (64, [1, 1, 3, 8, 1, 2]), (128, [5, 12, 7, 1, 9])])
def test_state_prefix(d, slots, decay, reverse, in_place):
    lens = [n * C - 5 * (i % 2) for i, n in enumerate(slots)]   # every second document ends inside a slot
    cu = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32)
    B, H = 2 if len(slots) == 1 else 1, 3   # (packed documents: one batch row)
    lam = np.array([0.5, 0.9, 1.0], np.float32) if decay else None
    p = bd.Problem(B, H, int(cu[-1]), d, C, C, "f32", cu if len(slots) > 1 else None, decay=lam)
    T = sum(slots)
    M = torch.randn(B, H, T, d, d, generator=torch.Generator().manual_seed(T * d + decay))
    want, at = torch.zeros_like(M, dtype=torch.float64), 0
    for n, length in zip(slots, lens):
        run = torch.zeros(B, H, d, d, dtype=torch.float64)
        for i in reversed(range(n)) if reverse else range(n):
            want[:, :, at + i] = run
            w = 1.0 if lam is None else torch.from_numpy(lam.astype(np.float64) ** min(C, length - i * C))[None, :, None, None]
            run = w * run + M[:, :, at + i].double()
        at += n
    src = M.cuda()
    got = src if in_place else torch.full_like(src, float("nan"))
    bd.lasp2_state_prefix(p, src, got, reverse)
    # at most T roundings of the running sum, 2^-24 each, and of the factor (its exponent rounds to fp32: 16 log2(0.5) * 2^-24)
    err = (got.cpu().double() - want).abs().max().item()
    assert err <= (T + 16) * 2.0 ** -24 * max(1.0, want.abs().max().item())


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("N", [1, 31, 257])
def test_softmax_row_sums(dtype, d, N):
    p = bd.Problem(1, 3, N, d, 64, 0, dtype)
    gen = torch.Generator(device="cuda").manual_seed(N * d)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dO = (torch.randn(1, 3, N, d, generator=gen, device="cuda").to(tdt) for _ in range(4))
    O, dQ, dK, dV = (torch.empty_like(Q) for _ in range(4))
    LSE = torch.empty(1, 3, N, device="cuda")
    ws = torch.full((bd.lasp2_softmax_workspace_size(p) // 4,), float("nan"), device="cuda")
    bd.lasp2_softmax_fwd(p, Q, K, V, O, LSE, True)
    bd.lasp2_softmax_bwd(p, Q, K, V, O, dO, LSE, dQ, dK, dV, ws, True)
    terms = (O.double() * dO.double()).view(-1, d)
    err = (ws[:3 * N].double() - terms.sum(1)).abs()   # the workspace begins with the row sums
    assert bool((err <= d * 2.0 ** -24 * terms.abs().sum(1)).all())   # d roundings of at most the sum of magnitudes
