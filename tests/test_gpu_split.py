"""fp32 products on the bf16 matrix cores (split operands): tile edges, k remainders, odd strides, values that the split
does not represent, and the packed operand against the one split in place."""
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
# three of them, k and row counts around multiples of 32, 128 and 256
SHAPES = [(70000, 255, 33), (33000, 257, 64), (30011, 1001, 61), (20001, 383, 81), (13001, 513, 97), (10007, 769, 128),
          (17000, 289, 129), (12001, 320, 145), (8003, 479, 176), (9001, 353, 289), (4999, 385, 383), (46000, 128, 128)]


@pytest.mark.parametrize("m,n,l", SHAPES)
@pytest.mark.parametrize("pad", [0, 1])
def test_products(m, n, l, pad):
    say("split products", m, n, l, pad)
    A = _randn(m, n, 1, pad)
    _check(ctx().rsvd_stage_gemm_an(A, _randn(n, l, 2, pad)), A, _randn(n, l, 2, pad))
    Q = _randn(m, l, 3, pad)
    _check(ctx().rsvd_stage_gemm_atn(A, Q), A.T, Q)


@pytest.mark.parametrize("l", [40, 160])
def test_values_outside_the_split(l):
    """Infinities, NaNs, values at the end of the range and tiles of nothing but tiny values."""
    import torch
    say("split extremes", l)
    m, n = 20000, 1024
    A, X = _randn(m, n, 4), _randn(n, l, 5) * 0.05
    A[7, 100] = float("inf")
    A[8, 101] = float("nan")
    A[300, 5] = -3.3e38
    A[301, 6] = 3.4e38
    A[512:1024] *= 1e-35
    A[1024:1536, ::2] = 0.0
    A[2048:2560, 256:512] *= 1e-33
    for got, want in ((ctx().rsvd_stage_gemm_an(A, X), A.double() @ X.double()),
                      (ctx().rsvd_stage_gemm_atn(A[:, :n], _randn(m, l, 6)), A.double().T.contiguous() @ _randn(m, l, 6).double())):
        want32 = want.float()
        assert bool((torch.isnan(got) == torch.isnan(want32)).all())
        inf = torch.isinf(want32)
        assert bool((got[inf] == want32[inf]).all())
        fine = torch.isfinite(want32)
        # row by row (the rows differ in scale by 70 decades): 1024 terms at most along a row of A X
        if got.shape[0] == m:
            err = torch.where(fine, (got - want).abs(), 0.0).amax(1)
            size = (torch.where(torch.isfinite(A), A, 0.0).double().norm(dim=1) * 0.05).clamp_min(1e-300)
            assert float((err / size).max()) <= 64 * EPS
    A = _randn(m, n, 7) * 1e-34                      # every tile takes the fp32 instruction
    rel = (ctx().rsvd_stage_gemm_an(A, X).double() - A.double() @ X.double()).norm() / (A.double() @ X.double()).norm()
    assert float(rel) <= 2 * np.sqrt(n) * EPS


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
