"""The small passes between the large kernels, against 64-bit sums.  Prefix and suffix of the states: where the
walk's batches of eight slots and the documents' borders meet (fewer slots than a batch, one more or less,
several documents in a batch).  Row sums of the softmax backward, by the
gradients they enter: every head size and type, numbers of rows beside those of a workgroup."""
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
@pytest.mark.parametrize("H", [15, 16])
@pytest.mark.parametrize("slots", [[8] * 5, [7] * 5, [1, 2, 9, 20, 8, 8] * 7, [3] * 70 + [40], [33]])
def test_documents_of_packed_batches_in_turn_and_by_marks(slots, H):
    """Prefix, suffix and total of packed states on both sides of the line between the two orders (16 groups and eight slots
    per document on average), with one, two and three documents per mark; the arrays' NaN must not reach a result."""
    lens = [n * C - 5 * (i % 2) for i, n in enumerate(slots)]
    cu, d, T = np.concatenate([[0], np.cumsum(lens)]).astype(np.int32), 32, sum(slots)
    p = bd.Problem(1, H, int(cu[-1]), d, C, C, "f32", cu)
    M = torch.randn(1, H, T, d, d, generator=torch.Generator(device="cuda").manual_seed(T + H), device="cuda")
    at = np.concatenate([[0], np.cumsum(slots)])
    part = [M[:, :, a:b].double() for a, b in zip(at[:-1], at[1:])]
    # at most 40 roundings of a document's running sum, 2^-24 each
    tol = lambda want: 40 * 2.0 ** -24 * max(1.0, want.abs().max().item())
    for reverse in (False, True):
        got = torch.full_like(M, float("nan"))
        bd.lasp2_state_prefix(p, M, got, reverse)
        want = torch.cat([(x.flip(2).cumsum(2).flip(2) if reverse else x.cumsum(2)) - x for x in part], 2)
        assert (got.double() - want).abs().max().item() <= tol(want)
    got = torch.full_like(M, float("nan"))
    bd.lasp2_state_total(p, M, got)
    want = torch.cat([x.sum(2, keepdim=True).expand_as(x) for x in part], 2)
    assert (got.double() - want).abs().max().item() <= tol(want)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("d", [16, 32, 64, 128])
@pytest.mark.parametrize("N", [1, 31, 257])
def test_softmax_row_sums(dtype, d, N):
    """dS = P (dP - delta), delta = dO . O: with an O of 64 times the usual size delta is most of dS, so dQ and dK carry its
    relative error (and that of the other terms) row by row."""
    p = bd.Problem(1, 3, N, d, 64, 0, dtype)
    gen = torch.Generator(device="cuda").manual_seed(N * d)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    Q, K, V, dO, O = (torch.randn(1, 3, N, d, generator=gen, device="cuda").to(tdt) for _ in range(5))
    dQ, dK, dV = (torch.empty_like(Q) for _ in range(3))
    LSE = torch.empty(1, 3, N, device="cuda")
    ws = torch.full((bd.lasp2_softmax_workspace_size(p) // 4,), float("nan"), device="cuda")
    bd.lasp2_softmax_fwd(p, Q, K, V, torch.empty_like(Q), LSE, True)
    O = O * 64
    bd.lasp2_softmax_bwd(p, Q, K, V, O, dO, LSE, dQ, dK, dV, ws, True)
    q, k, v, w, o = (x[0].double().cpu() for x in (Q, K, V, dO, O))
    tr = lambda x: x.transpose(1, 2).contiguous()
    P = torch.softmax((q @ tr(k) / d ** 0.5).masked_fill(torch.ones(N, N).triu(1).bool(), -float("inf")), 2)
    size = (w * o).abs().sum(2, keepdim=True)                    # what delta is the sum of
    ds = P * (w @ tr(v) - (w * o).sum(2, keepdim=True)) / d ** 0.5
    # Per row, against the row if every delta had the size of its terms: fp32 d 2^-24 for the sum and as much for the
    # rounded exponent (scores below 2^3) and the sums over N rows; bf16 2^-8 each for P, dS and the result.
    tol = (2 * d + N) * 2.0 ** -24 if dtype == "f32" else 3 * 2.0 ** -8
    big = P * size / d ** 0.5
    for name, got, want, scale in (("dQ", dQ, ds @ k, (big ** 2 @ (k ** 2)).sum(2)),
                                   ("dK", dK, tr(ds) @ q, (tr(big) ** 2 @ (q ** 2)).sum(2))):
        err = (got[0].double().cpu() - want).norm(dim=2)
        assert bool((err <= tol * scale.sqrt()).all()), (name, (err / scale.sqrt()).max().item(), tol)
