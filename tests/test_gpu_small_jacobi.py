"""Small SVD in one workgroup: sweeps, and the corrections of the whole matrix that take the place of the last ones."""
import ctypes as C

import numpy as np
import pytest
import torch

import parity
import workloads
from paper_2110_03423_amd import binding
from gpu_util import ctx, say, to_dev, to_np

pytestmark = pytest.mark.gpu

NPDT = {"f32": np.float32, "f64": np.float64}


def _matrix(l, kind, dt):
    i, rng = np.arange(l), np.random.default_rng(l)
    s = {"fast": np.exp(-3.0 * i / l), "slow": (1.0 + i) ** -0.1, "steep": 10.0 ** (-i / 8.0), "gauss": None, "tiny": 1e-15 / (1.0 + i),
         "clusters": np.where(i < l // 2, 1.0, 0.5) * (1 + 1e-6 * rng.random(l)),
         "half": np.where(i < l // 2, 1.0 + 1e-5 * rng.random(l), 0.9 ** (i - l // 2.0)), "rank": np.where(i < l - 5, 1.0 / (1 + i), 0.0)}[kind]
    if s is None:
        return np.linalg.qr(rng.standard_normal((l + 9, l)))[1].T.astype(NPDT[dt])
    near = np.linalg.qr(np.eye(l) + 0.05 * rng.standard_normal((l, l)))[0]      # nearly aligned, as a power iteration leaves them
    return np.linalg.qr((workloads.orthonormal_factor(l, l, 1) * s) @ near)[1].T.astype(NPDT[dt])


# orders on either side of a multiple of 16 (blocks of the products), the smallest and the largest with corrections, one beyond
@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [15, 16, 17, 31, 32, 33, 47, 48, 49, 63, 64, 65, 79, 80, 81])
@pytest.mark.parametrize("kind", ["fast", "slow", "steep", "gauss", "tiny", "clusters", "rank"])
def test_small_jacobi(dt, l, kind):
    say("small jacobi", dt, l, kind)
    M = _matrix(l, kind, dt)
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M))
    assert info.status == 0 and info.jacobi_sweeps <= 20
    sig, X, W = (to_np(t).astype(np.float64) for t in (sig, X, W))
    M64, eps, tol = M.astype(np.float64), np.finfo(NPDT[dt]).eps, parity.jacobi_tol(l, dt)
    want = np.linalg.svd(M64, compute_uv=False)
    say("  values", np.abs(sig - want).max() / want[0] / eps, "residual", np.linalg.norm(X * sig @ W.T - M64) / want[0] / tol)
    assert (np.diff(sig) <= 0).all() and np.abs(sig - want).max() <= 20 * eps * np.sqrt(l) * want[0]
    assert np.linalg.norm(X * sig @ W.T - M64) <= tol * want[0]
    # each column of W goes through ~l rotations a sweep: a random walk of ~20 l roundings; its length is set to one at the end: l / 16 + 4
    # roundings of its square, summed in fp64 by sixteen lanes (half of that for its length), one of the factor and one of the elements
    assert np.abs(W.T @ W - np.eye(l)).max() <= 8 * eps * np.sqrt(20 * l)
    length = np.sqrt((W.astype(np.longdouble) ** 2).sum(axis=0))
    if dt == "f32" or l <= 64:                     # (65 and more in fp64: the block kernels)
        assert np.abs(length - 1).max() <= 2 * eps + (l / 16 + 4) / 2 * 2.0 ** -52
    nz = sig > 100 * l * eps * want[0]
    # The rule that ends the sweeps takes the next one for granted where the last two converged by an order of 1.5: in an fp64 cluster of relative
    # width 1e-6 that one would still have found inner products of 1e-13 to 1e-12, with corrections or without.
    known = 1e-11 if kind == "clusters" and dt == "f64" else 0.0
    assert np.linalg.norm((X.T @ X)[np.ix_(nz, nz)] - np.eye(nz.sum())) <= tol + known


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [16, 33, 48, 64, 80])
def test_corrections_are_counted(dt, l):
    """jacobi_sweeps has the corrections in it: a sweep that turned by 1e-3 over the gap leaves what its own rotations moved, which is far above
    the threshold, and one sweep says nothing about a rate, so a second step of either kind follows."""
    say("corrections counted", dt, l)
    M = np.diag(np.linspace(2.0, 1.0, l)) + 1e-3 * workloads.gaussian_matrix(l, l, l)
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(M.astype(NPDT[dt])))
    say("  steps", info.jacobi_sweeps)
    assert info.status == 0 and 2 <= info.jacobi_sweeps <= 8


# (order, sweeps that the kernel without corrections takes)
CLUSTERED = [("f32", "half", {32: 5, 33: 5, 48: 5, 64: 5, 80: 4}), ("f32", "clusters", {32: 3, 33: 3, 48: 3, 64: 3, 80: 3}),
             ("f64", "half", {16: 6, 17: 7, 33: 7, 48: 8, 64: 8}), ("f64", "clusters", {16: 6, 17: 5, 33: 7, 48: 8, 64: 8})]


@pytest.mark.parametrize("dt,kind,l,sweeps", [(d, k, l, n) for d, k, c in CLUSTERED for l, n in c.items()])
def test_clusters_are_left_to_sweeps(dt, kind, l, sweeps):
    """Half of the values or more in clusters, where corrections of the whole matrix do not converge: they are not tried before they do, so there are
    no more steps than sweeps alone and the first correction behind a sweep that had nearly finished."""
    say("clusters", dt, kind, l)
    sig, X, W, info = ctx().rsvd_stage_jacobi(to_dev(_matrix(l, kind, dt)))
    say("  steps", info.jacobi_sweeps, "sweeps alone", sweeps)
    assert info.status == 0 and info.jacobi_sweeps <= sweeps + 1


@pytest.mark.parametrize("dt", ["f32", "f64"])
@pytest.mark.parametrize("l", [16, 48, 64])
def test_special_matrices(dt, l):
    """Nothing to rotate, equal columns, zero, values that are not finite (as they come out: no wait, no write elsewhere)."""
    c, T = ctx(), NPDT[dt]
    eps = np.finfo(T).eps
    d = np.linspace(2.0, 1.0, l).astype(T)
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(np.diag(d)))
    assert info.jacobi_sweeps == 1 and np.abs(to_np(sig) - d).max() <= 2 * eps
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(np.zeros((l, l), T)))
    assert info.status == 0 and not to_np(sig).any()
    one = np.ones((l, l), T)
    sig, X, W, info = c.rsvd_stage_jacobi(to_dev(one))
    sig, W = to_np(sig).astype(np.float64), to_np(W).astype(np.float64)
    assert info.status == 0 and abs(sig[0] - l) <= 20 * eps * l and sig[1] <= 20 * eps * l
    assert np.linalg.norm(W.T @ W - np.eye(l)) <= parity.jacobi_tol(l, dt)
    one[0, 0] = np.nan
    M, guard = to_dev(one), 512
    out = [torch.full((n + 2 * guard,), 7.0, dtype=M.dtype, device=M.device) for n in (l, l * l, l * l)]
    dtype, need, info = binding.F32 if dt == "f32" else binding.F64, C.c_size_t(), binding._Info()
    c._check(c.lib.rsvd_stage_workspace_bytes(c.h, dtype, l, l, C.byref(need)))
    ws = torch.full((need.value + 2 * 4096,), 7, dtype=torch.uint8, device=M.device)
    at = [C.c_void_p(t.data_ptr() + guard * t.element_size()) for t in out]
    c._check(c.lib.rsvd_stage_jacobi(c.h, c._stream(), dtype, l, C.c_void_p(M.data_ptr()), *at, C.c_void_p(ws.data_ptr() + 4096), need.value, C.byref(info)))
    for t in out:
        assert bool((t[:guard] == 7).all()) and bool((t[-guard:] == 7).all())
    assert bool((ws[:4096] == 7).all()) and bool((ws[-4096:] == 7).all())
    assert info.jacobi_sweeps <= 4                 # (the column with the NaN is left alone, the others are equal)
