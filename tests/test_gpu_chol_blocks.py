"""CholeskyQR: diagonal blocks whose pivots are all good, and blocks in which one is too small, at every place it can have."""
import numpy as np
import pytest

import parity
import workloads
from gpu_util import ctx, say, to_dev, to_np

pytestmark = pytest.mark.gpu

NPDT = {"f32": np.float32, "f64": np.float64}


# orders on either side of a multiple of 16 and of the orders with another distribution of the rows; the dependent column first but
# one, last, and on either side of the edge of a block
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [1, 2, 15, 16, 17, 33, 64, 65, 80, 96, 97, 113, 128, 140, 200])
@pytest.mark.parametrize("where", ["none", "second", "edge", "behind", "last"])
def test_dependent_columns(dt, l, where):
    at = {"none": None, "second": 1, "edge": 15, "behind": 16, "last": l - 1}[where]
    if at is not None and not 1 <= at < l:
        pytest.skip("no such column")
    say("dependent column", dt, l, where)
    rows, eps = 3 * l + 200, np.finfo(NPDT[dt]).eps
    Y = workloads.gaussian_matrix(rows, l, 50 + l).astype(NPDT[dt])
    if at is not None:
        Y[:, at] = Y[:, at - 1]
    Q, R, info = ctx().rsvd_stage_orth(to_dev(Y), want_r=True)
    Q, R = to_np(Q).astype(np.float64), to_np(R)
    say("  raised", info.raised_pivots, "refilled", info.refilled_columns)
    assert info.status == 0
    # (a duplicate of a column is left at the rounding of the panel: replaced in fp32, set aside in fp64 and replaced or resolved behind)
    assert info.refilled_columns + info.raised_pivots == 0 if at is None else info.refilled_columns + info.raised_pivots >= 1
    # as for the other panels of these tests: two rounds leave a few roundings in each product of two columns, l of them in the norm
    assert parity.orthonormality(Q) <= 10 * l * eps
    # a column of Y goes through two triangular solves of order l, each with an error of order l eps of its norm in the worst case
    assert np.linalg.norm(Y - Q @ R) <= 50 * l * eps * np.linalg.norm(Y)
    assert l == 1 or np.abs(np.tril(R, -1)).max() == 0.0
