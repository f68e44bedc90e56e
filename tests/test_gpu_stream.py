"""Narrow products with A^T that read A straight into the matrix instructions: remainders of rows, columns and k, every number of column
blocks and of wavefronts to a tile, rows of any alignment, infinities, batches."""
import numpy as np
import pytest

from gpu_util import ctx, say

pytestmark = pytest.mark.gpu

EPS = {"f32": 2.0 ** -23, "f64": 2.0 ** -52}


def _randn(dt, shape, seed, pad=0):
    """N(0, 1) on the GPU; pad > 0: a view with that many columns of NaN in front (unaligned, longer rows)."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    X = torch.randn(*shape[:-1], shape[-1] + pad, dtype=torch.float64, device="cuda:0", generator=g)
    X[..., :pad] = float("nan")
    return X.to(torch.float32 if dt == "f32" else torch.float64)[..., pad:]


def _check(dt, got, A, Q):
    """Each of K additions rounds a partial sum s_k by at most eps / 2 of it: a random walk of errors eps / sqrt(12) |s_k|, and s_k is one of sqrt(k)
    products, so that the standard deviation is 0.2 eps K products' root mean square.  Allowed is twenty times that (the
    walk of a sum that is large throughout is five times the usual one, and an fp64 reference has as much): no element of a million is off by it,
    but a single term is far above it."""
    A, Q = A.double().T.contiguous(), Q.double().contiguous()
    K, want = A.shape[1], A @ Q
    bound = 4 * EPS[dt] * K ** 0.5 * ((A * A) @ (Q * Q)).sqrt()
    worst = float(((got.double() - want).abs() / bound).max())
    say("  worst", worst)
    assert worst <= 1
    # (the bound itself: a result without its last k, or of zeros, is not within it; one whose last tile of rows is missing has rows of zeros)
    last = A[:, -1][:, None] * Q[-1][None, :]
    assert not bool((last.abs() <= bound).all()) and bool((want.abs() > bound).any(dim=1).all())


# (rows of A = k, columns of A = rows of the result, l), a million entries of A and more, which this kernel takes: one, two and three column
# blocks; tiles of 64 rows with 1 to 63 left over; k ranges with remainders of steps, of turns and of groups; one and many ranges; queues
# of a CU with one, two and more workgroups; results with fewer rows than a lane reads
SHAPES = [(262147, 4, 4), (200003, 5, 3), (110003, 65, 16), (16001, 66, 17), (17003, 67, 31), (4003, 257, 32), (30011, 191, 1),
          (1021, 1024, 16), (33, 40001, 32), (31, 33000, 18), (5001, 2003, 30), (2500, 5000, 15), (1200, 22000, 20), (9001, 4099, 9),
          (3003, 1001, 33), (7001, 515, 47), (2002, 3001, 48), (61, 20483, 40), (40960, 256, 32), (25536, 1232, 18), (304, 6528, 24), (241, 4783, 38)]


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("m,n,l", SHAPES)
def test_products(dt, pad, m, n, l):
    say("stream products", dt, pad, m, n, l)
    A, Q = _randn(dt, (m, n), 1, pad), _randn(dt, (m, l), 2, pad)
    _check(dt, ctx().rsvd_stage_gemm_atn(A, Q), A, Q)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,n,l", [(4003, 301, 17), (20001, 67, 32)])
def test_infinities_stay(dt, m, n, l):
    """An infinity meets nothing but its own column of A and row of Q, in the last k as well (k that do not exist are zero on both sides)."""
    import torch
    say("stream infinities", dt, m, n, l)
    A, Q = _randn(dt, (m, n), 3), _randn(dt, (m, l), 4)
    A[m - 1, n - 1] = float("inf")
    Q[m - 1, 0] = float("-inf")
    got = ctx().rsvd_stage_gemm_atn(A, Q)
    assert bool(torch.isfinite(got[: n - 1, 1:]).all())
    assert bool((got[n - 1, 1:] == torch.sign(Q[m - 1, 1:]) * float("inf")).all())
    assert bool((got[: n - 1, 0] == -torch.sign(A[m - 1, : n - 1]) * float("inf")).all())


@pytest.mark.parametrize("dt,batch,m,n,k,p", [("f32", 5, 901, 501, 20, 11), ("f32", 40, 500, 260, 10, 6), ("f64", 3, 1000, 403, 20, 20), ("f64", 17, 333, 300, 8, 8)])
def test_problems_of_a_batch(dt, batch, m, n, k, p):
    """Each problem of a batch gives what a call of its own gives (other ranges of k: to rounding)."""
    import torch
    say("stream batch", dt, batch, m, n, k, p)
    U, V = np.linalg.qr(np.random.default_rng(5).standard_normal((m, 60)))[0], np.linalg.qr(np.random.default_rng(6).standard_normal((n, 60)))[0]
    base = torch.from_numpy((U * 0.8 ** np.arange(60)) @ V.T).to("cuda:0", torch.float32 if dt == "f32" else torch.float64)
    A = torch.stack([torch.roll(base, 7 * b, 0) * (1.0 + b) for b in range(batch)]).contiguous()
    S, U, Vt, info = ctx().rsvd_run_batched(A, k=k, p=p, q=1, seed=3)
    assert info.status == 0
    for b in (0, batch - 1):
        s, u, vt, _ = ctx().rsvd_run(A[b], k=k, p=p, q=1, seed=3 + b)
        # (values to 50 eps of the largest; a vector moves by eps over its gap, here 0.2 s_j at least: s_1 / s_j as many times more)
        assert float((S[b] - s).abs().max() / s[0]) <= 50 * EPS[dt]
        d = 1.0 - (Vt[b] * vt).sum(1).abs()
        assert bool((d.double() <= (200 * EPS[dt] * float(s[0]) / s.double()) + 8 * EPS[dt]).all())
