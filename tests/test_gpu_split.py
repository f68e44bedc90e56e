"""fp32 products on the bf16 matrix cores (split operands): tile edges, k remainders, odd strides, values of every size and
beyond the range, and the packed operand against the one split in place."""
import numpy as np
import pytest

from gpu_util import ctx, say

pytestmark = pytest.mark.gpu

EPS = 2.0 ** -23


def _randn(rows, cols, seed, pad=0):
    """rows x cols N(0, 1) fp32 on the GPU; pad > 0: a view with that many columns in front (unaligned, longer rows)."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    return torch.randn(rows, cols + pad, device="cuda:0", generator=g)[:, pad:]


def _check(got, A, X):
    """Any summation order of exact products stays within K eps sum |a b|, element by element; the norm-wise error of the
    two-level sums grows like sqrt(K / 32) roundings of the result."""
    K = A.shape[1]
    A, X = A.double().contiguous(), X.double().contiguous()
    want = A @ X
    bound = K * EPS * (A.abs() @ X.abs()) + 1e-300
    assert bool(((got.double() - want).abs() <= bound).all())
    rel = float((got.double() - want).norm() / want.norm())
    assert rel <= (2.0 + np.sqrt(K / 32.0)) * EPS, rel


# each with at least 2^29 multiply-adds, below which the fp32 instruction is used: column tiles of 48 to 144, one to
# three of them, k and row counts around multiples of 32, 128 and 256; the second half fills the chip in both directions and with both
# kinds of loads, so that every instance of the kernel is reached
SHAPES = [(70000, 255, 33), (33000, 257, 64), (30011, 1001, 61), (20001, 383, 81), (13001, 513, 97), (10007, 769, 128),
          (17000, 289, 129), (12001, 320, 145), (8003, 479, 176), (9001, 353, 289), (4999, 385, 383), (46000, 128, 128),
          (30000, 1024, 48), (60000, 500, 60), (15000, 1504, 80), (11000, 1600, 96), (21000, 600, 112), (40001, 333, 129),
          (18003, 640, 176), (24000, 700, 210), (15000, 1052, 380), (9004, 1004, 288), (12001, 1032, 160)]


@pytest.mark.parametrize("m,n,l", SHAPES)
@pytest.mark.parametrize("pad", [0, 1])
def test_products(m, n, l, pad):
    say("split products", m, n, l, pad)
    A = _randn(m, n, 1, pad)
    _check(ctx().rsvd_stage_gemm_an(A, _randn(n, l, 2, pad)), A, _randn(n, l, 2, pad))
    Q = _randn(m, l, 3, pad)
    _check(ctx().rsvd_stage_gemm_atn(A, Q), A.T, Q)


def _by_rows(got, A, X, roundings, slack=2.0 ** -143):
    """Element by element, where the result is finite: that many roundings of sum |a b|, whatever the row's size (slack: 64
    roundings of partial sums in the subnormal range)."""
    import torch
    A, X = A.double().contiguous(), X.double().contiguous()
    want, size = A @ X, A.abs() @ X.abs()
    w32 = want.float()
    assert bool((torch.isnan(got) == torch.isnan(w32)).all())
    inf = torch.isinf(w32)
    assert bool((got[inf] == w32[inf]).all())
    fine = torch.isfinite(w32)
    err = (got.double() - want).abs()[fine]
    assert bool((err <= roundings * 0.5 * EPS * size[fine] + slack).all())


@pytest.mark.parametrize("l", [40, 128, 160])
@pytest.mark.parametrize("pad", [0, 1])
@pytest.mark.parametrize("top", [0, 90, 127])
def test_every_value_passes_through(l, pad, top):
    """Products with columns of the identity give back what was put in, bit for bit: fp32 numbers of every size side by side, from
    the smallest subnormal up to 2^top (2^96 and above: the workgroup computes its tile again)."""
    import torch
    say("split identity", l, pad, top)
    m, n = 20000, 1056
    A = _randn(m, n + pad, 4)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(5)
    A = torch.ldexp(A, torch.randint(-149, top - 3, (m, n + pad), device="cuda:0", generator=g).float())[:, pad:]
    cols, rows = torch.arange(l, device="cuda:0") * 5 % n, torch.arange(l, device="cuda:0") * 97 % m
    X, Q = torch.zeros(n, l, device="cuda:0"), torch.zeros(m, l, device="cuda:0")
    X[cols, torch.arange(l)] = 1.0
    Q[rows, torch.arange(l)] = 1.0
    assert bool((ctx().rsvd_stage_gemm_an(A, X) == A[:, cols]).all())
    assert bool((ctx().rsvd_stage_gemm_atn(A, Q) == A[rows].T).all())


@pytest.mark.parametrize("l", [40, 112, 160])
def test_rows_of_any_size(l):
    """Rows of 1e-37 beside ordinary ones, and a block of 1e-36 that ends inside the tiles."""
    say("split rows", l)
    m, n = 20000, 1024
    A, X, Q = _randn(m, n, 4), _randn(n, l, 5), _randn(m, l, 6)
    A[::7] *= 1e-37
    A[3000:3333, 100:933] *= 1e-36
    A[:, 5::11] *= 1e-5
    for _ in range(2):
        # one rounding per k-tile of 32 and those inside one
        _by_rows(ctx().rsvd_stage_gemm_an(A, X), A, X, n // 32 + 48)
        _by_rows(ctx().rsvd_stage_gemm_atn(A, Q), A.T, Q, m // 32 + 48)
        A *= 1e-34                                    # (rows of zeros and subnormal numbers among them)


@pytest.mark.parametrize("l", [40, 128, 160])
def test_values_outside_the_split(l):
    """Infinities, NaNs, values and results at the end of the range: the rest of such a tile is right as well."""
    import torch
    say("split extremes", l)
    m, n = 20000, 1024
    A, X, Q = _randn(m, n, 4), _randn(n, l, 5) * 0.05, _randn(m, l, 6)
    A[7, 100] = float("inf")
    A[8, 101] = float("nan")
    A[300, 5] = -3.3e38
    A[301, 6] = 3.4e38
    A[512:1024] *= 1e-35
    A[1024:1536, ::2] = 0.0
    A[5000:5100] *= 1e33
    _by_rows(ctx().rsvd_stage_gemm_an(A, X), A, X, 2 * n)              # (any order of summation)
    _by_rows(ctx().rsvd_stage_gemm_atn(A, Q), A.T, Q, 2 * m)
    # products just below the largest number: their leading parts alone are above it
    big = 1.8446e19
    A = torch.full((m, n), big, device="cuda:0")
    cols = torch.arange(l, device="cuda:0") * 5 % n
    X, Q = torch.zeros(n, l, device="cuda:0"), torch.zeros(m, l, device="cuda:0")
    X[cols, torch.arange(l)] = -big
    Q[cols, torch.arange(l)] = big
    assert bool((ctx().rsvd_stage_gemm_an(A, X) == (A[0, 0] * -A[0, 0])).all())
    assert bool((ctx().rsvd_stage_gemm_atn(A, Q) == (A[0, 0] * A[0, 0])).all())
    assert bool(torch.isfinite(A[0, 0] * A[0, 0]))


# column tiles of 80 to 144, two and three of them; at 6000 x 1500, l = 280 and 20000 x 5000, l = 140 tiles of up to 128 columns, which
# would do without the packed operand, would lead to other k ranges
@pytest.mark.parametrize("m,n,k,p,q", [(6000, 1500, 150, 20, 1), (2000, 9001, 190, 11, 2), (6000, 1500, 256, 24, 1),
                                       (20000, 5000, 130, 10, 1), (9001, 2203, 129, 0, 1), (12000, 3000, 400, 30, 0)])
def test_without_room_for_the_packed_operand(m, n, k, p, q):
    """A workspace that lacks it is still accepted and gives the same bits."""
    import torch
    say("no packed operand", m, n, k)
    c = ctx()
    A = (_randn(m, 300, 8) * torch.exp(-torch.arange(300, device="cuda:0") / 60.0)) @ _randn(300, n, 9)
    need = c.workspace_bytes(0, m, n, k, p, q)
    full, less = (torch.empty(b, dtype=torch.uint8, device="cuda:0") for b in (need, need - 256))
    a = c.rsvd_run(A, k, p, q, workspace=full)
    b = c.rsvd_run(A, k, p, q, workspace=less)
    assert a[3].status == 0 and b[3].status == 0
    for x, y in zip(a[:3], b[:3]):
        assert bool((x == y).all())


def _low_rank(m, n, r, seed, batch=None):
    """r singular values from 1 down to 0.05, exact to fp32 rounding."""
    import torch
    g = torch.Generator(device="cuda:0")
    g.manual_seed(seed)
    lead = () if batch is None else (batch,)
    U = torch.linalg.qr(torch.randn(*lead, m, r, dtype=torch.float64, generator=g, device="cuda:0").cpu())[0].cuda()
    V = torch.linalg.qr(torch.randn(*lead, n, r, dtype=torch.float64, generator=g, device="cuda:0").cpu())[0].cuda()
    s = torch.logspace(0, np.log10(0.05), r, dtype=torch.float64, device="cuda:0")
    return (torch.matmul((U * s).float(), V.transpose(-1, -2).float().contiguous())).contiguous()


def _reconstructs(A, S, U, Vt):
    """All of A lies in the k triplets: what is left is the rounding of A, of the factors and of k-term sums, and none of the values
    is off by more than the norm of that."""
    left = float((A.double() - (U.double() * S.double()) @ Vt.double()).norm() / A.double().norm())
    assert left <= 16 * EPS * np.sqrt(U.shape[1]), left
    I = np.eye(U.shape[1])
    for B in (U.double().T.contiguous() @ U.double(), Vt.double() @ Vt.double().T.contiguous()):
        assert np.abs(B.cpu().numpy() - I).max() <= 16 * EPS * np.sqrt(U.shape[1])


# column tiles of 48, 96, 112, 128 and 144 (packed in both directions), odd sizes and 16-byte rows, k remainders of 3 to 32
@pytest.mark.parametrize("m,n,k,p", [(40011, 1003, 30, 10), (30003, 1205, 80, 16), (20001, 1600, 100, 12), (20000, 1600, 100, 28),
                                     (12001, 2203, 129, 8), (12000, 2208, 130, 10)])
def test_centered(m, n, k, p):
    """The column means are taken away while A is split."""
    import torch
    say("split centred", m, n, k, p)
    A = _low_rank(m, n, k - 1, m)
    A -= A.mean(0)
    g = torch.Generator(device="cuda:0")
    g.manual_seed(n)
    A += 0.01 * torch.randn(n, device="cuda:0", generator=g)          # (twice the size of the entries)
    S, U, Vt, info, mean = ctx().rsvd_run_centered(A, k, p, 1, seed=5)
    assert info.status == 0
    mu = A.double().mean(0)
    assert float((mean.double() - mu).abs().max()) <= 2 * EPS * float(mu.abs().max())
    C = (A.double() - mu).float()
    left = float((C.double() - (U.double() * S.double()) @ Vt.double()).norm() / C.double().norm())
    # rounding of A, larger than C by |mu|, and of the factors
    assert left <= (16 * np.sqrt(k) + 2 * float(A.double().norm() / C.double().norm())) * EPS, left


@pytest.mark.parametrize("batch,m,n,k,p", [(24, 2003, 501, 30, 10), (16, 3000, 1000, 80, 16), (9, 2001, 1203, 100, 28), (3, 9000, 640, 48, 16)])
def test_batched(batch, m, n, k, p):
    say("split batch", batch, m, n, k, p)
    A = _low_rank(m, n, k, batch, batch)
    S, U, Vt, info = ctx().rsvd_run_batched(A, k, p, 1, seed=5)
    assert info.status == 0
    for b in range(batch):
        _reconstructs(A[b], S[b], U[b], Vt[b])
        one = ctx().rsvd_run(A[b].contiguous(), k, p, 1, seed=5 + b)[0]
        assert float(((S[b] - one) / one).abs().max()) <= 64 * EPS


# A width that is no multiple of four leaves the workspace's panels unaligned; the fp32 kernel reads them in 16-byte pieces all the same, but
# is the less exact of the two.  Short k ranges, narrow outputs and last waves that are nearly empty are where it would be taken otherwise.
@pytest.mark.parametrize("m,n,l,k", [(68683, 130, 112, 102), (100000, 130, 120, 45), (40001, 260, 200, 77), (90000, 240, 160, 43)])
def test_products_of_odd_width_stay_split(m, n, l, k):
    """U = Q W of a whole call: Q is what the call leaves in the first panel of its workspace, W follows from U and Q (the roundings of m rows
    average out), and what is left are the roundings of the product: those of the stage call, which has no slack behind its operands, with
    the same Q and W.  The fp32 kernel's are 2.8 to 5 times as large."""
    import torch
    say("odd lift", m, n, l, k)
    A = _randn(m, n, 9) * torch.exp(-torch.arange(n, device="cuda:0") * (2.0 / n))
    c = ctx()
    ws = torch.empty(c.workspace_bytes(0, m, n, k, l - k, 0), dtype=torch.uint8, device="cuda:0")
    U = c.rsvd_run(A, k, l - k, 0, seed=4, workspace=ws)[1]
    Q = ws[: m * l * 4].view(torch.float32).view(m, l).clone()
    Q64 = Q.double()
    Qt = Q64.T.contiguous()
    W = torch.linalg.solve(Qt @ Q64, Qt @ U.double()).float().contiguous()
    exact = Q64 @ W.double()
    run, stage = (float((x.double() - exact).norm() / exact.norm()) for x in (U, c.rsvd_stage_lift(Q, W, k)))
    say("  errors", run, stage)
    assert run <= 1.5 * stage, (run, stage)
