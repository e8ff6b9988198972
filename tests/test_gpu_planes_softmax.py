"""Causal softmax attention on the split planes with two mirrored row tiles per workgroup: the shorter tile's waves fill the stages of
the longer one once they are done.  Lengths on both sides of a tile of 32, of a stage (32 rows of partners for each share) and of
two, where no stage, one or many are left for them; a middle tile with no mirror image; shares of the queries, whose shorter
tile is long too; non-finite keys and values in a stage that one of the tiles sees.  Against the definition in 64 bits, tile
by tile."""
import pytest
import torch

from paper_2502_07563_amd import binding as bd
from tests.util import TOL

pytestmark = pytest.mark.gpu


def _inputs(G, N, d, dtype, seed):
    gen = torch.Generator(device="cuda").manual_seed(seed)
    tdt = torch.float32 if dtype == "f32" else torch.bfloat16
    return [torch.randn(1, G, N, d, generator=gen, device="cuda").to(tdt) for _ in range(4)]


def _run(p, x, n=None, q0=0):
    Q, K, V, dO = x
    n = n or Q.shape[2]
    Q, dO = Q[:, :, q0:q0 + n].contiguous(), dO[:, :, q0:q0 + n].contiguous()
    O, lse = torch.empty_like(Q), torch.empty(Q.shape[:3], dtype=torch.float32, device="cuda")
    grads = [torch.empty_like(t) for t in (Q, K, V)]
    ws = torch.empty(bd.lasp2_softmax_workspace_size(p) // 4, dtype=torch.float32, device="cuda")
    if n == x[0].shape[2]:
        bd.lasp2_softmax_fwd(p, Q, K, V, O, lse, True)
        bd.lasp2_softmax_bwd(p, Q, K, V, O, dO, lse, *grads, ws, True)
    else:
        bd.lasp2_softmax_fwd_share(p, q0, n, Q, K, V, O, lse, True)
        bd.lasp2_softmax_bwd_share(p, q0, n, Q, K, V, O, dO, lse, *grads, ws, True)
    return [O] + grads


def _want(x, n, q0):
    q, k, v, w = (t[0].double() for t in x)
    q, w = q[:, q0:q0 + n], w[:, q0:q0 + n]
    i = torch.arange(q0, q0 + n, device="cuda")
    s = q @ k.transpose(1, 2).contiguous() * q.shape[2] ** -0.5
    s = s.masked_fill(torch.arange(k.shape[1], device="cuda")[None] > i[:, None], float("-inf"))
    p = s.softmax(2)
    o = p @ v
    ds = p * (w @ v.transpose(1, 2).contiguous() - (w * o).sum(2, keepdim=True)) * q.shape[2] ** -0.5
    return [o, ds @ k, ds.transpose(1, 2).contiguous() @ q, p.transpose(1, 2).contiguous() @ w]


def _check(got, want, dtype, what):
    for name, a, b in zip(("O", "dQ", "dK", "dV"), got, want):
        a = a[0].double()
        # a tile's rows against their own size, or what the smallest have: a hundredth of the tensor's mean
        floor = b.norm() / b.shape[1] ** 0.5 * 32 ** 0.5 / 100
        for r in range(0, b.shape[1], 32):
            err = ((a[:, r:r + 32] - b[:, r:r + 32]).norm() / torch.maximum(b[:, r:r + 32].norm(), floor)).item()
            assert err <= TOL[dtype], (name, r, err, what)


CASES = [("f32", 64), ("f32", 128), ("f32", 16), ("f32", 32), ("bf16", 64), ("bf16", 32), ("bf16", 16)]


@pytest.mark.parametrize("dtype,d", CASES)
def test_lengths(dtype, d):
    for N in (32, 33, 64, 65, 96, 127, 129, 161, 192, 255, 257, 320, 321, 383, 450, 513, 640, 769, 1100):
        p = bd.Problem(1, 2, N, d, 64, 0, dtype)
        x = _inputs(2, N, d, dtype, N)
        _check(_run(p, x), _want(x, N, 0), dtype, (N, d))


@pytest.mark.parametrize("dtype,d", CASES)
def test_shares(dtype, d):
    for N, q0, n in ((700, 300, 400), (700, 0, 130), (513, 480, 33), (1000, 100, 31), (900, 255, 257)):
        p = bd.Problem(1, 2, N, d, 64, 0, dtype)
        x = _inputs(2, N, d, dtype, N)
        _check(_run(p, x, n, q0), _want(x, n, q0), dtype, (N, q0, n))


@pytest.mark.parametrize("dtype,d", CASES)
def test_what_is_not_finite_stays_where_it_belongs(dtype, d):
    """A NaN in one row of V or K: the rows before it are those without it, the rows from it on are NaN, where it is the last, the
    first or a middle row of a stage, of the sequence, or lies in the part that the longer tile alone sees."""
    N = 457
    p = bd.Problem(1, 2, N, d, 64, 0, dtype)
    for which in (1, 2):
        for j in (0, 31, 128, 255, 300, 455, 456):
            x = _inputs(2, N, d, dtype, j)
            want = _want(x, N, 0)
            x[which][0, 1, j, 3] = float("nan")
            O, dQ = _run(p, x)[:2]
            assert torch.isnan(O[0, 1, j:]).any(dim=1).all() and torch.isnan(dQ[0, 1, j:]).any(dim=1).all(), (which, j)
            for a, b in ((O, want[0]), (dQ, want[1])):
                for h, rows in ((0, N), (1, j)):
                    if rows:
                        err = ((a[0, h, :rows].double() - b[h, :rows]).norm() / b[h].norm()).item()
                        assert err <= TOL[dtype], (which, j, h, err)
