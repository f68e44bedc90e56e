"""GPU parity, stage by stage: every step of Algorithm 1 through the C ABI
against the CPU oracle on the same seeded inputs."""
import numpy as np
import pytest

import workloads
from oracle import philox as ophilox
from oracle import rsvd as orc
from oracle import jacobi as ojacobi
import parity
from gpu_util import ctx, to_dev, to_np, say

pytestmark = pytest.mark.gpu

NPDT = {"f32": np.float32, "f64": np.float64}
CODE = {"f32": 0, "f64": 1}


# ---------------------------------------------------------------- step 1: sketch
def test_philox_raw_bit_exact():
    c = ctx()
    for seed, first, n in ((0, 0, 1 << 20), (0x0123456789ABCDEF, (1 << 32) - 500, 1000), (7, 12345, 1)):
        say("philox raw", seed, first, n)
        got = to_np(c.rsvd_stage_philox_raw(seed, first, n)).view(np.uint32)
        want = ophilox.philox_groups(seed, first, n)
        assert (got == want).all()
    got = to_np(c.rsvd_stage_philox_raw(3, 10, 64, stream_id=5)).view(np.uint32)
    assert (got == ophilox.philox_groups(3, 10, 64, stream=5)).all()


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("shape", [(2000, 80), (1001, 21), (1, 1), (3, 5)])
def test_sketch_matches_oracle(dt, shape):
    say("sketch", dt, shape)
    n, l = shape
    got = to_np(ctx().rsvd_stage_sketch(11, n, l, CODE[dt])).astype(np.float64)
    want = ophilox.philox_normal(11, n, l, NPDT[dt]).astype(np.float64)
    # fp32: both sides round one fp64 value, so they differ by at most one fp32 ulp where the
    # fp64 libm results straddle a rounding boundary.  fp64: log, sqrt, sincos and two
    # multiplications, each within ~1-2 ulp on either side -> 8 eps relative.
    eps = np.finfo(NPDT[dt]).eps
    tol = (1.0 if dt == "f32" else 8.0) * eps * np.maximum(1.0, np.abs(want))
    assert (np.abs(got - want) <= tol).all()
    if dt == "f32":
        assert (got != want).mean() < 1e-3


def test_sketch_strided_and_empty():
    import torch
    c = ctx()
    buf = torch.full((50, 16), -7.0, dtype=torch.float64, device="cuda:0")
    c.rsvd_stage_sketch(2, 50, 10, 1, out=buf[:, :10])
    got = to_np(buf)
    want = ophilox.philox_normal(2, 50, 10, np.float64)
    np.testing.assert_allclose(got[:, :10], want, rtol=1e-14, atol=1e-15)
    assert (got[:, 10:] == -7.0).all()
    assert c.rsvd_stage_sketch(2, 0, 10, 1).shape == (0, 10)


# ---------------------------------------------------------------- steps 2, 4, 6: products
GEMM_CASES = [
    # m, n, l : several tiles with ragged tails, vector and scalar load paths, split-K shapes
    (333, 517, 20), (1000, 260, 80), (130, 4100, 16), (4100, 130, 24), (257, 129, 21),
    (96, 64, 64), (700, 300, 120), (5000, 100, 100), (64, 9000, 48), (513, 515, 7),
]


def _gemm_check(got, A, X, K, dt):
    want = A @ X
    eps = np.finfo(NPDT[dt]).eps
    bound = K * eps * (np.abs(A) @ np.abs(X)) + 1e-300      # rigorous: any summation order
    assert (np.abs(got - want) <= bound).all(), float(np.max(np.abs(got - want) / bound))
    rel = np.linalg.norm(got - want) / np.linalg.norm(want)
    assert rel <= 4 * np.sqrt(K) * eps, rel
    return rel


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,n,l", GEMM_CASES)
def test_range_product(dt, m, n, l):
    say("gemm_an", dt, m, n, l)
    A = workloads.gaussian_matrix(m, n, 1, NPDT[dt])
    X = workloads.gaussian_matrix(n, l, 2, NPDT[dt])
    got = to_np(ctx().rsvd_stage_gemm_an(to_dev(A), to_dev(X))).astype(np.float64)
    _gemm_check(got, A.astype(np.float64), X.astype(np.float64), n, dt)


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,n,l", GEMM_CASES)
def test_adjoint_product(dt, m, n, l):
    say("gemm_atn", dt, m, n, l)
    A = workloads.gaussian_matrix(m, n, 3, NPDT[dt])
    X = workloads.gaussian_matrix(m, l, 4, NPDT[dt])
    got = to_np(ctx().rsvd_stage_gemm_atn(to_dev(A), to_dev(X))).astype(np.float64)
    _gemm_check(got, A.astype(np.float64).T, X.astype(np.float64), m, dt)


def test_products_with_leading_dimensions():
    import torch
    A = workloads.gaussian_matrix(300, 200, 5, np.float32)
    X = workloads.gaussian_matrix(200, 40, 6, np.float32)
    Abig = torch.zeros((300, 212), dtype=torch.float32, device="cuda:0")
    Abig[:, :200] = to_dev(A)
    Xbig = torch.zeros((200, 44), dtype=torch.float32, device="cuda:0")
    Xbig[:, :40] = to_dev(X)
    got = to_np(ctx().rsvd_stage_gemm_an(Abig[:, :200], Xbig[:, :40])).astype(np.float64)
    _gemm_check(got, A.astype(np.float64), X.astype(np.float64), 200, "f32")


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("m,l,k,tr", [(1000, 80, 64, False), (517, 20, 10, True), (2000, 120, 100, True),
                                      (130, 33, 7, False)])
def test_lift(dt, m, l, k, tr):
    say("lift", dt, m, l, k, tr)
    Q = workloads.gaussian_matrix(m, l, 7, NPDT[dt])
    W = workloads.gaussian_matrix(l, l, 8, NPDT[dt])
    got = to_np(ctx().rsvd_stage_lift(to_dev(Q), to_dev(W), k, transpose_out=tr)).astype(np.float64)
    if tr:
        got = got.T
    _gemm_check(got, Q.astype(np.float64), W.astype(np.float64)[:, :k], l, dt)


# ---------------------------------------------------------------- step 3: orthonormalisation
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("rows,l,cond", [(512, 20, 10.0), (3000, 80, 1e3), (1000, 120, 50.0), (129, 33, 5.0),
                                         (10000, 64, 1e2), (2000, 160, 30.0), (3000, 288, 1e2), (5000, 576, 10.0),
                                         (1500, 200, 1e3), (2500, 900, 10.0)])     # 900: past the strip inverse's LDS limit
def test_orth_full_rank_matches_householder(dt, rows, l, cond):
    say("orth", dt, rows, l, cond)
    Y = workloads.graded_matrix(rows, l, cond, seed=20, dtype=NPDT[dt])
    Qg, Rg, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Qg, Rg = to_np(Qg).astype(np.float64), to_np(Rg)
    Qo, Ro = orc.qr_positive(Y.astype(np.float64))
    eps = np.finfo(NPDT[dt]).eps
    assert info.refilled_columns == 0 and info.status == 0
    assert parity.orthonormality(Qg) <= 10 * l * eps
    # the positive-diagonal QR is unique; CholeskyQR2 reaches it to ~eps * cond
    assert np.abs(Qg - Qo).max() <= 20 * eps * cond
    assert np.abs(Rg - Ro).max() <= 20 * eps * cond * np.abs(Ro).max()
    assert np.abs(np.tril(Rg, -1)).max() == 0.0


@pytest.mark.parametrize("rows,l,cond", [(2000, 48, 1e9), (1500, 96, 1e11), (3000, 160, 1e10), (800, 20, 1e8),
                                         (4000, 288, 1e9)])
def test_orth_ill_conditioned_fp64_panel_matches_householder(rows, l, cond):
    """fp64 panels whose singular values span far more than the six decades one CholeskyQR round resolves (the
    paper's step 3 is a Householder QR, which keeps every direction down to the rounding level): the raised
    pivots of the first round and the additional round must deliver the same Q and R, with no column replaced."""
    say("orth ill-conditioned", rows, l, cond)
    Y = workloads.graded_matrix(rows, l, cond, seed=21, dtype=np.float64)
    Qg, Rg, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Qg, Rg = to_np(Qg), to_np(Rg)
    Qo, Ro = orc.qr_positive(Y)
    eps = np.finfo(np.float64).eps
    say("  raised", info.raised_pivots, "refilled", info.refilled_columns)
    assert info.status == 0 and info.refilled_columns == 0 and info.raised_pivots > 0
    assert parity.orthonormality(Qg) <= 10 * l * eps
    assert np.linalg.norm(Y - Qg @ Rg) <= 50 * l * eps * np.linalg.norm(Y)
    assert np.abs(np.tril(Rg, -1)).max() == 0.0
    # Householder QR itself fixes column j of Q only to eps * (cond of the leading j columns); compare at that level
    assert np.abs(Qg - Qo).max() <= 50 * eps * cond
    assert np.abs(Rg - Ro).max() <= 50 * eps * cond * np.abs(Ro).max()


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_orth_rank_deficient_input(dt):
    """rank 10 < l = 20 (the situation of the planted rank-10 configuration)."""
    say("orth rank deficient", dt)
    rows, l, r = 512, 20, 10
    B = workloads.gaussian_matrix(rows, r, 30) @ workloads.gaussian_matrix(r, l, 31)
    Y = B.astype(NPDT[dt])
    Qg, Rg, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Qg, Rg = to_np(Qg).astype(np.float64), to_np(Rg)
    eps = np.finfo(NPDT[dt]).eps
    say("  refilled", info.refilled_columns)
    assert parity.orthonormality(Qg) <= 10 * l * eps
    Y64 = Y.astype(np.float64)
    # range(Q) contains range(Y), and Y = Q R
    assert np.linalg.norm(Y64 - Qg @ (Qg.T @ Y64)) <= 50 * l * eps * np.linalg.norm(Y64)
    assert np.linalg.norm(Y64 - Qg @ Rg) <= 50 * l * eps * np.linalg.norm(Y64)
    if dt == "f64":
        assert info.refilled_columns == l - r


def test_orth_zero_and_nonfinite_input():
    import torch
    Y = torch.zeros((100, 8), dtype=torch.float64, device="cuda:0")
    Q, _, info = ctx().rsvd_stage_orth(Y)
    assert info.refilled_columns == 8
    assert parity.orthonormality(to_np(Q)) <= 1e-13
    Y = to_dev(workloads.gaussian_matrix(100, 8, 1))
    Y[5, 3] = float("nan")
    from paper_2110_03423_amd import RsvdError
    with pytest.raises(RsvdError) as ei:
        ctx().rsvd_stage_orth(Y)
    assert ei.value.code == 1


# ---------------------------------------------------------------- step 5: small SVD
def _svd_check(sig, X, W, M, dt, name):
    l = M.shape[0]
    tol = parity.jacobi_tol(l, dt)
    want = np.linalg.svd(M, compute_uv=False)
    smax = want[0]
    assert np.abs(sig - want).max() <= tol * smax, (name, np.abs(sig - want).max())
    assert (np.diff(sig) <= 0).all()
    assert np.linalg.norm(W.T @ W - np.eye(l)) <= tol
    nz = sig > 100 * l * np.finfo(NPDT[dt]).eps * smax
    assert np.linalg.norm((X.T @ X)[np.ix_(nz, nz)] - np.eye(nz.sum())) <= tol
    assert np.linalg.norm(X * sig @ W.T - M) <= tol * smax


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [2, 5, 20, 33, 64, 80, 96, 128, 129, 160, 200, 288, 333, 576])
def test_jacobi_matches_oracle(dt, l):
    say("jacobi", dt, l)
    M = workloads.gaussian_matrix(l, l, 40 + l, NPDT[dt])
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M))
    sig, X, W = (to_np(t).astype(np.float64) for t in (sig, X, W))
    say("  sweeps", info.jacobi_sweeps)
    assert info.status == 0 and 1 <= info.jacobi_sweeps <= 20
    M64 = M.astype(np.float64)
    _svd_check(sig, X, W, M64, dt, "gaussian")
    # every column goes through ~l rotations per sweep: their rounding errors must add up like a random walk
    # (a rotation whose c^2 + s^2 is off by a few 1e-8 in the same direction every time shows up here)
    want = np.linalg.svd(M64, compute_uv=False)
    assert np.abs(sig - want).max() <= 20 * np.finfo(NPDT[dt]).eps * np.sqrt(l) * want[0]
    if l <= 33:       # brute-force Jacobi oracle on the small ones: vectors up to sign
        Xo, so, Wo, _ = ojacobi.jacobi_svd(M64)
        tol = 1e3 * np.finfo(NPDT[dt]).eps / np.min(np.abs(np.diff(so)) / so[:-1]) if l > 1 else 1
        assert np.abs(np.abs(np.sum(X * Xo, axis=0)) - 1).max() <= min(0.1, tol)
        assert np.abs(np.abs(np.sum(W * Wo, axis=0)) - 1).max() <= min(0.1, tol)


# The blocked factorisation cuts l into blocks of 96, or of 112 and 128 where that makes one less: the first and the last order of each choice,
# last blocks of one column, of one more and one less than 16, and whole ones; a column that depends on others in a late block.
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [192, 193, 209, 224, 225, 240, 241, 256, 257, 288, 289, 337, 384, 385])
def test_orthonormalize_blocked(dt, l):
    say("blocked factorisation", dt, l)
    rows = 2 * l + 17
    Y = workloads.gaussian_matrix(rows, l, l, NPDT[dt])
    Y[:, l - 2] = Y[:, 5] - Y[:, l // 2]
    Q, R, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Q, R = to_np(Q).astype(np.float64), to_np(R)
    eps = np.finfo(NPDT[dt]).eps
    assert info.status == 0 and info.refilled_columns >= 1
    # as for the small panels; the condition of a Gaussian panel of twice as many rows is below 10
    assert np.abs(Q.T @ Q - np.eye(l)).max() <= 16 * eps * np.sqrt(l)
    assert np.abs(np.tril(R, -1)).max() == 0
    norms = np.linalg.norm(Y.astype(np.float64), axis=0)
    assert (np.linalg.norm(Q @ R - Y, axis=0) <= (64 * np.sqrt(l) * eps) * norms.max()).all()


# The product of the rounds' triangular factors: strips of 16 columns, wavefronts of up to five 16-row blocks, groups of 640 rows and what is left of
# them, orders whose inverse no longer goes by strips.  In fp64 the dependent column adds the factors of the additional rounds.
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [18, 33, 127, 128, 129, 639, 640, 641, 657, 1296])
def test_triangular_factor_of_all_rounds(dt, l):
    say("product of the factors", dt, l)
    Y = workloads.gaussian_matrix(2 * l + 17, l, l + 1, NPDT[dt])
    Y[:, l - 2] = Y[:, 5] - Y[:, l // 2]
    Q, R, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Q, R = to_np(Q).astype(np.float64), to_np(R)
    assert info.status == 0 and info.refilled_columns >= 1
    assert np.abs(np.tril(R, -1)).max() == 0
    norms = np.linalg.norm(Y.astype(np.float64), axis=0)      # bound as for the blocked factorisation above
    assert (np.linalg.norm(Q @ R - Y, axis=0) <= (64 * np.sqrt(l) * np.finfo(NPDT[dt]).eps) * norms.max()).all()


# fp64 products of 16-byte rows go through a ring of k-tiles in LDS: every column tile, one row and one k more and less than tiles of 64, 128
# and 16, one k-tile in all, several k ranges with an uneven last one, outputs of two and three column tiles; each of the five tiles for more
# than 128 columns in either direction.
@pytest.mark.parametrize("m,n,l", [(64, 16, 16), (66, 18, 10), (62, 4098, 30), (4098, 62, 32), (1026, 1000, 48), (1000, 1030, 50), (130, 3002, 66),
                                   (2050, 514, 96), (514, 2050, 98), (700, 900, 112), (902, 700, 128), (1298, 640, 130), (640, 1310, 192),
                                   (1154, 1026, 290), (20002, 302, 20), (2800, 2630, 162), (4778, 782, 382), (8288, 478, 286), (2100, 3570, 260),
                                   (2050, 1026, 194), (3644, 2876, 280)])
def test_fp64_products(m, n, l):
    say("fp64 products", m, n, l)
    rng = np.random.default_rng(m + n + l)
    A, X, Q = rng.standard_normal((m, n)), rng.standard_normal((n, l)), rng.standard_normal((m, l))
    c, eps = ctx(), np.finfo(np.float64).eps
    for got, want, a, b in ((c.rsvd_stage_gemm_an(to_dev(A), to_dev(X)), A @ X, A, X), (c.rsvd_stage_gemm_atn(to_dev(A), to_dev(Q)), A.T @ Q, A.T, Q)):
        # partial sums of up to |a_i| |b_j| / sqrt(terms), whose roundings add up like a random walk over the terms, on either side: eps |a_i| |b_j|; 8:
        # the largest of up to 1e6
        size = np.linalg.norm(a, axis=1)[:, None] * np.linalg.norm(b, axis=0)[None, :]
        assert (np.abs(to_np(got) - want) <= 8 * eps * size).all()


# Of the Gram matrix of an fp64 panel of more than 128 columns only the tiles on or above the diagonal are computed: long panels, whose rows are
# cut into ranges with an uneven last one.  An error of the second round's Gram matrix is one of Q^T Q.
@pytest.mark.parametrize("rows,l", [(5003, 130), (3001, 290), (20001, 256), (9000, 144)])
def test_fp64_gram_of_long_panels(rows, l):
    say("fp64 gram", rows, l)
    Y = workloads.gaussian_matrix(rows, l, l, np.float64)
    Q, R, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Q, R, eps = to_np(Q), to_np(R), np.finfo(np.float64).eps
    assert info.status == 0 and info.refilled_columns == 0 and info.raised_pivots == 0
    assert np.abs(Q.T @ Q - np.eye(l)).max() <= 16 * eps * np.sqrt(l)          # (bounds as for the blocked factorisation)
    assert np.abs(np.tril(R, -1)).max() == 0
    assert (np.linalg.norm(Q @ R - Y, axis=0) <= (64 * np.sqrt(l) * eps) * np.linalg.norm(Y, axis=0).max()).all()


# The last k-tile of a product whose k range is no multiple of 16 is filled up with what does not count, whatever it is: infinite results
# stay infinite, in the rows where an operand is and nowhere else.
@pytest.mark.parametrize("m,n,l", [(1002, 1000, 32), (998, 1004, 130)])
def test_fp64_products_with_infinities(m, n, l):
    import torch
    say("fp64 infinities", m, n, l)
    rng = np.random.default_rng(l)
    A, X, Q = rng.uniform(0.5, 1.5, (m, n)), rng.uniform(0.5, 1.5, (n, l)), rng.uniform(0.5, 1.5, (m, l))
    kx, kq = (n - 1) // 16 * 16, (m - 1) // 16 * 16       # where the last k-tile begins, for A X and for A^T Q
    c = ctx()
    for place in ("a", "b"):
        B, Y, Z = A.copy(), X.copy(), Q.copy()
        if place == "a":
            B[5, kx], B[kq, 7] = np.inf, -np.inf
        else:
            Y[kx, 3], Z[kq, l - 1] = np.inf, -np.inf
        for got, want in ((c.rsvd_stage_gemm_an(to_dev(B), to_dev(Y)), B @ Y), (c.rsvd_stage_gemm_atn(to_dev(B), to_dev(Z)), B.T @ Z)):
            got, fine = to_np(got), np.isfinite(want)
            assert (got[~fine] == want[~fine]).all()
            assert np.abs(got[fine] - want[fine]).max() <= 4 * max(m, n) * np.finfo(np.float64).eps * 1.5 * 1.5


# Rounding errors of a product grow with the number of terms that go into one accumulator.  The kernel for operands of 16-byte rows may cut
# the k range into fewer pieces than the one for others, but not add up longer chains: same matrices, one element further on in memory.
@pytest.mark.parametrize("m,n,l", [(3000, 20000, 16), (5000, 5000, 64), (20000, 10000, 96), (400, 50000, 100), (6000, 6000, 128),
                                   (8000, 12000, 288), (12000, 9000, 262)])
def test_fp64_products_add_up_no_longer_chains(m, n, l):
    import torch
    say("fp64 chains", m, n, l)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(m + n + l)

    def whole(rows, cols):           # whole numbers of up to 29 bits, in two pieces whose products and sums are exact
        x = (torch.randn(rows, cols, dtype=torch.float64, device="cuda:0", generator=g) * 2.0 ** 26).round().clamp(-2.0 ** 29, 2.0 ** 29)
        hi = torch.floor(x / 32768.0)
        return x, hi, x - hi * 32768.0

    def shifted(x):
        y = torch.empty(x.shape[0], x.shape[1] + 1, dtype=x.dtype, device=x.device)[:, 1:]
        y.copy_(x)
        return y

    def error(got, a, b):
        hh, mid, ll = a[1] @ b[1], a[1] @ b[2] + a[2] @ b[1], a[2] @ b[2]
        return float((((got - hh * 2.0 ** 30) - mid * 32768.0) - ll).norm() / got.norm())

    A, X, Q = whole(m, n), whole(n, l), whole(m, l)
    At = tuple(x.T.contiguous() for x in A)
    c = ctx()
    for f, a, b in ((c.rsvd_stage_gemm_an, A, X), (c.rsvd_stage_gemm_atn, At, Q)):
        one, other = error(f(A[0], b[0]), a, b), error(f(shifted(A[0]), b[0]), a, b)
        say("  errors", one, other)
        assert one <= 1.05 * other


# Small fp32 panels are orthonormalised in one workgroup up to 16 columns and 1024 rows: one column, rows that are no multiple of
# 16, the largest panel, the first ones beyond, and columns that depend on others (replaced, the same either way).
@pytest.mark.parametrize("rows,l,rank", [(1, 1, 1), (17, 1, 1), (40, 16, 16), (333, 7, 7), (1024, 16, 16), (1025, 16, 16), (1024, 17, 17),
                                         (500, 13, 9), (64, 16, 15), (1001, 15, 8), (777, 6, 3), (1024, 16, 14)])
def test_orthonormalize_small_panels(rows, l, rank):
    say("small panel", rows, l, rank)
    c = ctx()
    Y = workloads.gaussian_matrix(rows, l, 3, np.float32)
    Y[:, rank:] = Y[:, :l - rank]
    D = to_dev(np.concatenate([Y, np.ones((rows, 3), np.float32)], axis=1))[:, :l]          # a leading dimension of l + 3
    Q, R, info = c.rsvd_stage_orth(D, want_r=True)
    Q, R = to_np(Q).astype(np.float64), to_np(R)
    eps = np.finfo(np.float32).eps
    assert info.status == 0 and info.refilled_columns >= l - rank
    # Q^T Q: sums of `rows` products of entries rounded to eps, the rounding errors adding up like a random walk
    assert np.abs(Q.T @ Q - np.eye(l)).max() <= 16 * eps * np.sqrt(l)
    assert np.abs(np.tril(R, -1)).max(initial=0) == 0
    # Y = Q R: a round is a product with R^-1 rounded to eps, l terms (condition below 10 here); what a dependent column leaves
    # behind lies below the pivot threshold, 32 eps of its norm
    norms = np.linalg.norm(Y, axis=0)
    assert (np.linalg.norm(Q @ R - Y, axis=0) <= (64 * np.sqrt(l) * eps) * norms.max()).all()


# One task per block pair of 16-column blocks: the smallest orders, an odd number of blocks (one sits out every step), a last block of
# one and of fifteen columns, the longest columns that the panel in LDS holds and the first order beyond it (column by column).
@pytest.mark.parametrize("dt,l", [("f64", 97), ("f64", 113), ("f64", 127), ("f64", 464), ("f64", 465), ("f32", 129), ("f32", 145),
                                  ("f32", 255), ("f32", 1088), ("f32", 1089)])
def test_block_jacobi_edges(dt, l):
    say("block jacobi", dt, l)
    M = workloads.graded_matrix(l, l, 1e3, seed=l, dtype=NPDT[dt])
    M[:, 3] = 0                                   # a column that is never rotated
    c = ctx()
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(M))
    assert info.status == 0 and info.jacobi_sweeps <= 20
    again = c.rsvd_stage_jacobi(to_dev(M))        # whichever workgroup took which task
    for a, b in zip((sig, X, W), again[:3]):
        assert np.array_equal(to_np(a), to_np(b))
    sig, X, W = (to_np(t).astype(np.float64) for t in (sig, X, W))
    _svd_check(sig, X, W, M.astype(np.float64), dt, "graded")
    # each of the l columns of W has length 1 up to a random walk of ~20 l roundings
    eps = np.finfo(NPDT[dt]).eps
    assert np.abs(np.linalg.norm(W, axis=0) - 1).max() <= 4 * eps * np.sqrt(20 * l)


# What the corrections of the whole matrix behind the sweeps meet: angles of every size (each length of the series, halvings), clusters
# that they leave to further sweeps, zero and negligible columns; orders with one and with 31 rows or columns in the last 32 x 32 tile,
# and on either side of a limit on the angles.  The first four are the smallest and largest orders that would fit into one workgroup.
@pytest.mark.parametrize("dt,l", [("f64", 65), ("f64", 96), ("f32", 97), ("f32", 128), ("f64", 97), ("f64", 159), ("f64", 257), ("f32", 129), ("f32", 161), ("f32", 191), ("f32", 290)])
@pytest.mark.parametrize("kind", ["fast", "slow", "steep", "clusters", "rank"])
def test_block_jacobi_corrections(dt, l, kind):
    say("block jacobi corrections", dt, l, kind)
    i = np.arange(l)
    rng = np.random.default_rng(l)
    s = {"fast": np.exp(-3.0 * i / l), "slow": (1.0 + i) ** -0.1, "steep": 10.0 ** (-i / 12.0),
         "clusters": np.where(i < l // 2, 1.0, 0.5) * (1 + 1e-6 * rng.random(l)), "rank": np.where(i < l - 40, 1.0 / (1 + i), 0.0)}[kind]
    # nearly aligned factors, as a power iteration leaves them
    near = np.linalg.qr(np.eye(l) + 0.02 * rng.standard_normal((l, l)))[0]
    M = np.linalg.qr((workloads.orthonormal_factor(l, l, 1) * s) @ near)[1].T.astype(NPDT[dt])
    c = ctx()
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(M))
    assert info.status == 0
    again = c.rsvd_stage_jacobi(to_dev(M))        # whichever workgroup took which tile
    for a, b in zip((sig, X, W), again[:3]):
        assert np.array_equal(to_np(a), to_np(b))
    sig, X, W = (to_np(t).astype(np.float64) for t in (sig, X, W))
    M64, eps = M.astype(np.float64), np.finfo(NPDT[dt]).eps
    _svd_check(sig, X, W, M64, dt, kind)
    # a correction is exp of an antisymmetric matrix, orthogonal to a rounding or two per element: a random walk of ~20 l roundings over
    # sweeps and corrections, as for the lengths of the columns above
    assert np.abs(W.T @ W - np.eye(l)).max() <= 8 * eps * np.sqrt(20 * l)
    want = np.linalg.svd(M64, compute_uv=False)
    assert np.abs(sig - want).max() <= 20 * eps * np.sqrt(l) * want[0]


# Matrices in general position with steep spectra, whose columns do not show their grading, take more sweeps than others; the limit is 60 on one
# workgroup and in the one-launch block kernel.
@pytest.mark.parametrize("l", [56, 66, 72, 80, 89, 96, 97, 110])
@pytest.mark.parametrize("decades", [8.5, 11, 12])
def test_jacobi_takes_the_sweeps_it_needs(l, decades):
    say("jacobi many sweeps", l, decades)
    M = (workloads.orthonormal_factor(l, l, 1) * 10.0 ** (-np.arange(l) * decades / l)) @ workloads.orthonormal_factor(l, l, 2).T
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M))
    say("  sweeps", info.jacobi_sweeps)
    assert info.status == 0 and info.jacobi_sweeps <= 60
    sig, W = to_np(sig), to_np(W)
    tol = parity.jacobi_tol(l, "f64")
    assert np.abs(sig - np.linalg.svd(M, compute_uv=False)).max() <= tol and np.linalg.norm(W.T @ W - np.eye(l)) <= tol
    assert np.linalg.norm(to_np(X) * sig @ W.T - M) <= tol


# Many equal values above a decaying rest: angles below the threshold of a rotation, rounding noise each, are most of what a correction
# turns by, and its series has to be long enough for them.  Factors as q subspace iterations leave them.
@pytest.mark.parametrize("dt,l,equal,q,rate", [("f64", 70, 40, 2, 0.02), ("f64", 98, 90, 1, 0.05), ("f64", 110, 64, 2, 0.4), ("f64", 128, 96, 2, 0.05),
                                               ("f64", 160, 96, 0, 0.2), ("f64", 160, 96, 1, 0.02), ("f64", 200, 180, 0, 0.1),
                                               ("f64", 288, 100, 1, 0.02), ("f32", 110, 64, 2, 0.4), ("f32", 160, 96, 1, 0.05)])
def test_block_jacobi_equal_values(dt, l, equal, q, rate):
    say("block jacobi equal values", dt, l, equal, q, rate)
    rng = np.random.default_rng(1000 * l + equal + q)
    i = np.arange(l + 20)
    s = np.where(i < equal, 1.0, 0.8 * np.exp(-rate * np.maximum(i - equal, 0)))
    U, V = (np.linalg.qr(rng.standard_normal((2 * l, l + 20)))[0] for _ in range(2))
    A = (U * s) @ V.T
    Q = np.linalg.qr(A @ rng.standard_normal((2 * l, l)))[0]
    for _ in range(q):
        Q = np.linalg.qr(A @ np.linalg.qr(A.T @ Q)[0])[0]
    M = np.linalg.qr(A.T @ Q)[1].T.astype(NPDT[dt])
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M))
    assert info.status == 0
    sig, X, W = (to_np(t).astype(np.float64) for t in (sig, X, W))
    M64, eps = M.astype(np.float64), np.finfo(NPDT[dt]).eps
    _svd_check(sig, X, W, M64, dt, "equal values")
    assert np.abs(W.T @ W - np.eye(l)).max() <= 8 * eps * np.sqrt(20 * l)          # bounds as for the corrections above
    want = np.linalg.svd(M64, compute_uv=False)
    assert np.abs(sig - want).max() <= 20 * eps * np.sqrt(l) * want[0]


@pytest.mark.parametrize("l", [129, 300, 576])
@pytest.mark.parametrize("cond", [1.0, 1e3])
def test_block_jacobi_values_do_not_drift(l, cond):
    """The rotations of a visit are accumulated in fp64 and rounded once, and so are the columns: a random walk of two roundings per
    visit of a column block, blocks x sweeps of them (rotations in fp32 shrink or stretch a column the same way every time: 8, 20 and 33
    eps at these orders)."""
    say("block jacobi values", l, cond)
    M = workloads.gaussian_matrix(l, l, l, np.float32) if cond == 1.0 else workloads.graded_matrix(l, l, cond, seed=l, dtype=np.float32)
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M))
    want = np.linalg.svd(M.astype(np.float64), compute_uv=False)
    # relative to the value where it is resolved in fp32, else to what a rounding of the columns moves it by
    err = (to_np(sig).astype(np.float64) - want) / np.maximum(want, want[0] * 1e-2)
    eps = np.finfo(np.float32).eps
    bound = 0.5 * eps * np.sqrt(-(-l // 16) * info.jacobi_sweeps)
    assert info.status == 0
    assert np.sqrt(np.mean(err ** 2)) <= bound and abs(np.mean(err)) <= bound / 2


def test_block_jacobi_on_two_streams():
    """Two decompositions share the chip: neither waits for workgroups of its own that are not running yet."""
    import torch
    say("block jacobi on two streams")
    M = [to_dev(workloads.gaussian_matrix(288, 288, 70 + i)) for i in range(2)]
    c = [ctx(), type(ctx())()]
    want = [c[0].rsvd_stage_jacobi(m.clone())[:3] for m in M]
    torch.cuda.synchronize()
    streams = [torch.cuda.Stream() for _ in range(2)]
    got = [[], []]
    args = [[m.clone() for _ in range(3)] for m in M]
    torch.cuda.synchronize()
    for rep in range(3):
        for i in range(2):
            with torch.cuda.stream(streams[i]):
                got[i].append(c[i].rsvd_stage_jacobi(args[i][rep])[:3])
    torch.cuda.synchronize()
    for i in range(2):
        for g in got[i]:
            for a, b in zip(g, want[i]):
                assert np.array_equal(to_np(a), to_np(b))


@pytest.mark.parametrize("dt", ["f32", "f64"])
def test_jacobi_special_matrices(dt):
    say("jacobi special", dt)
    c = ctx()
    T = NPDT[dt]
    eps = np.finfo(T).eps
    d = np.array([3.0, 0.5, 7.0, 1.0, 0.0, 2.0])
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(np.diag(d).astype(T)))
    np.testing.assert_allclose(to_np(sig), np.sort(d)[::-1], rtol=4 * eps, atol=0)
    assert info.jacobi_sweeps == 1
    Q = workloads.orthonormal_factor(24, 24, 5).astype(T)
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(Q))
    np.testing.assert_allclose(to_np(sig), np.ones(24), rtol=50 * eps)
    u, v = workloads.gaussian_matrix(16, 1, 1), workloads.gaussian_matrix(16, 1, 2)
    M = (u @ v.T).astype(T)
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(M))
    sig = to_np(sig).astype(np.float64)
    assert sig[0] == pytest.approx(np.linalg.norm(u) * np.linalg.norm(v), rel=50 * eps)
    assert (sig[1:] <= 50 * eps * sig[0]).all()
    G = workloads.graded_matrix(32, 32, 1e6 if dt == "f64" else 1e3, seed=9, dtype=T)
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(G))
    _svd_check(*(to_np(t).astype(np.float64) for t in (sig, X, W)), G.astype(np.float64), dt, "graded")


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("n,l", [(256, 20), (2000, 80), (1000, 120), (300, 33), (2000, 288), (1000, 160)])
def test_small_svd_of_projected_factor(dt, n, l):
    say("small_svd", dt, n, l)
    Bt = workloads.graded_matrix(n, l, 100.0, seed=50, dtype=NPDT[dt])
    sig, Ub, V, info = ctx().rsvd_stage_small_svd(to_dev(Bt))
    sig, Ub, V = (to_np(t).astype(np.float64) for t in (sig, Ub, V))
    B = Bt.astype(np.float64).T
    Uo, so, Vto = orc.small_svd(B)
    eps = np.finfo(NPDT[dt]).eps
    tol = parity.jacobi_tol(l, dt)
    assert np.abs(sig - so).max() <= tol * so[0]
    assert np.linalg.norm(Ub * sig @ V.T - B) <= tol * so[0]
    assert parity.orthonormality(V) <= tol and parity.orthonormality(Ub) <= tol
    # graded spectrum 1 .. 1/100 in l steps: relative gaps ~ ln(100)/l, vectors well defined
    gap = np.log(100.0) / l
    assert np.abs(np.abs(np.sum(Ub * Uo, axis=0)) - 1).max() <= 100 * l * eps / gap
    assert np.abs(np.abs(np.sum(V * Vto.T, axis=0)) - 1).max() <= 100 * l * eps / gap


HARD_FACTORS = [  # (dtype, n, l, singular values of B): steep decays and flat clusters, orders on both Jacobi paths
    ("f32", 900, 96, lambda i, l: 10.0 ** (-i / 16.0), 12),                      # six decades
    ("f32", 1200, 261, lambda i, l: 10.0 ** (-i / 40.0), 12),                    # six and a half, block path
    ("f64", 800, 60, lambda i, l: 10.0 ** (-i / 5.0), 12),                       # twelve decades
    ("f64", 1000, 200, lambda i, l: 10.0 ** (-i / 20.0), 12),                    # ten, block path
    # flat clusters: inside one the sweeps gain a constant factor only, down to the rounding level of the type
    ("f32", 900, 80, lambda i, l: np.where(i < l // 2, 1.0, 1e-3), 12),
    ("f64", 1100, 200, lambda i, l: np.where(i < l // 2, 1.0, 1e-3), 20),
    ("f64", 700, 120, lambda i, l: np.where(i < l // 4, 10.0 ** (-i / 5.0), 1e-6), 20),   # a steep head above a flat tail
]


@pytest.mark.parametrize("dt,n,l,spec,max_sweeps", HARD_FACTORS,
                         ids=[f"{c[0]}-{c[1]}x{c[2]}-{j}" for j, c in enumerate(HARD_FACTORS)])
def test_small_svd_of_steep_and_clustered_factors(dt, n, l, spec, max_sweeps):
    """B with a steep spectrum or with clusters of equal singular values, in general position (no power iteration
    has lined its rows up): the rotations act on the rows of the triangular factor of B^T, which are graded like
    the singular values, and need about as many sweeps as on an easy factor (on its columns they needed 20 and
    more, or ran into the sweep cap); inside a cluster the vectors come out orthogonal to the rounding level."""
    say("small_svd hard", dt, n, l)
    T = NPDT[dt]
    i = np.arange(l, dtype=np.float64)
    s = np.asarray(spec(i, l), dtype=np.float64) * np.ones(l)
    B = (workloads.orthonormal_factor(l, l, 70) * s) @ workloads.orthonormal_factor(n, l, 71).T
    Bt = np.ascontiguousarray(B.T.astype(T))
    sig, Ub, V, info = ctx().rsvd_stage_small_svd(to_dev(Bt))
    sig, Ub, V = (to_np(t).astype(np.float64) for t in (sig, Ub, V))
    B = Bt.astype(np.float64).T
    so = np.linalg.svd(B, compute_uv=False)
    tol = parity.jacobi_tol(l, dt)
    say("  sweeps", info.jacobi_sweeps)
    assert info.status == 0 and info.jacobi_sweeps <= max_sweeps, info.jacobi_sweeps
    assert np.abs(sig - so).max() <= tol * so[0]
    big = so > so[0] * (1e-5 if dt == "f32" else 1e-10)
    assert (np.abs(sig - so)[big] / so[big]).max() <= (1e-3 if dt == "f32" else 1e-5)
    assert np.linalg.norm(Ub * sig @ V.T - B) <= tol * so[0]
    # singular values at the rounding level of the whole factor count as zero: their columns of Ub are zero
    live = so > 4 * np.finfo(T).eps * np.linalg.norm(so)
    assert parity.orthonormality(V) <= tol and parity.orthonormality(Ub[:, live]) <= tol
    assert all(np.abs(np.linalg.norm(Ub[:, j]) - 1) <= tol or not Ub[:, j].any() for j in np.where(~live)[0])


def test_small_svd_rank_deficient_factor():
    say("small_svd rank deficient")
    n, l, r = 256, 20, 10
    B = (workloads.gaussian_matrix(l, r, 60) @ workloads.gaussian_matrix(r, n, 61))
    sig, Ub, V, info = ctx().rsvd_stage_small_svd(to_dev(np.ascontiguousarray(B.T)))
    sig, Ub, V = (to_np(t) for t in (sig, Ub, V))
    so = np.linalg.svd(B, compute_uv=False)
    np.testing.assert_allclose(sig[:r], so[:r], rtol=1e-11)
    assert (sig[r:] <= 1e-12 * so[0]).all()
    assert np.linalg.norm(Ub[:, :r] * sig[:r] @ V[:, :r].T - B) <= 1e-12 * so[0]


def test_argument_errors_are_reported():
    import torch
    from paper_2110_03423_amd import RsvdError
    c = ctx()
    A = torch.zeros((10, 6), dtype=torch.float64, device="cuda:0")
    for k, p, q in ((0, 2, 1), (3, -1, 1), (3, 2, -1), (5, 2, 0)):
        with pytest.raises(RsvdError) as ei:
            c.rsvd_run(A, k, p, q, workspace=torch.zeros(1 << 20, dtype=torch.uint8, device="cuda:0"))
        assert ei.value.code < 0
    with pytest.raises(RsvdError) as ei:
        c.rsvd_run(A, 2, 2, 1, workspace=torch.zeros(256, dtype=torch.uint8, device="cuda:0"))
    assert ei.value.code == -19
