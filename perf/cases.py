"""The calls whose speed this repository is held to.

Every case is one call of the randomized SVD as a program makes it through the package's public class: the matrix is
on the GPU, the context is kept from call to call (and with it the workspace that its binding caches), the
outputs are allocated by the call.  Sizes are those of `workloads.py`, of `bench.py` and of the tests, and plain ones
between them.  `api` names the entry point:

  run       rsvd_run           one matrix
  centered  rsvd_run_centered  principal components of a data matrix, rows = observations
  batched   rsvd_run_batched   many matrices of one shape

A is a planted spectrum (orthonormal factors) plus a little noise, as in `workloads.py`.  Singular vectors are
defined up to sign; as a program does that follows its components from one call to the next, `run` turns them so
that they point along a basis it already has (`ref`).
"""
import math

import numpy as np
import torch

from paper_2110_03423_amd import JOB_S, JOB_SUV, JOB_SV, Rsvd

JOBS = {"S": JOB_S, "SV": JOB_SV, "SUV": JOB_SUV}
SKETCH_SEED = 7


def _case(name, api, dtype, m, n, k, p, q, job, law, rate, rank, noise, batch=1, info=False):
    """law "exp": s_i = exp(-rate i); "power": s_i = (1 + i)^-rate.  rank: planted values.  noise: standard deviation."""
    c = dict(api=api, dtype=dtype, m=m, n=n, k=k, p=p, q=q, job=job, law=law, rate=rate, rank=rank, noise=noise,
             batch=batch, info=info)
    return dict(c, name=name) if name else c


def listed():
    return [
        # an interactive call on a small table, status checked: launches and the small serial kernels are all of it;
        # rank 10 under a sketch of 20 columns, so the basis has to be completed
        _case("small f64", "run", "f64", 512, 256, 10, 10, 2, "SUV", "exp", math.log(10.0) / 5, 10, 0.0, info=True),
        # singular values only of a small block, as a rank test inside a larger program does it
        _case("values f32", "run", "f32", 300, 200, 8, 8, 1, "S", "exp", 0.25, 24, 1e-4),
        # the planted-spectrum benchmark of the paper at its usual size
        _case("bench f32", "run", "f32", 10000, 2000, 64, 16, 2, "SUV", "exp", -math.log(0.9), 2000, 0.0),
        # a table whose row length is odd, with the customary p = 10: nothing is a multiple of anything
        _case("ragged f32", "run", "f32", 30011, 2999, 51, 10, 2, "SUV", "exp", 0.06, 90, 1e-5),
        # more columns than rows, l above the orders that one workgroup solves
        _case("wide f32", "run", "f32", 4001, 50021, 200, 10, 1, "SV", "exp", 0.015, 315, 1e-5),
        # principal components of 100000 images of 1000 pixels
        _case("pca f32", "centered", "f32", 100000, 1000, 100, 20, 3, "SV", "power", 0.5, 200, 1e-4),
        # the paper's own 2000 x n experiments: fp64, slow decay, k = n / 10
        _case("paper f64", "run", "f64", 2000, 1000, 100, 10, 2, "SUV", "power", 0.1, 1000, 0.0),
        # a large dense fp64 operator
        _case("large f64", "run", "f64", 20000, 20000, 256, 32, 2, "SUV", "power", 1.0, 2048, 1e-6),
        # a large fp32 operator: the matrix cores' regime
        _case("large f32", "run", "f32", 65536, 16384, 512, 64, 1, "SUV", "exp", 1.0 / 128, 768, 1e-6),
        # a handful of leading directions of the same matrix: the memory's regime
        _case("leading f32", "run", "f32", 65536, 16384, 10, 6, 1, "SV", "exp", 0.2, 24, 1e-6),
        # clustering many data blocks: one call for all of them
        _case("batch f32", "batched", "f32", 2000, 500, 16, 16, 1, "SUV", "exp", 0.1, 48, 1e-5, batch=256),
        _case("batch f64", "batched", "f64", 4000, 1000, 32, 16, 2, "SUV", "exp", 0.06, 72, 1e-6, batch=32),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """Another call of the same ranges: up to 2^30 entries of A, up to l = 576 (128 in a batch), never dearer than the
    largest listed case of its precision."""
    while True:
        api = rng.choice(["run", "run", "run", "centered", "batched"])
        dtype = rng.choice(["f32", "f32", "f64"])
        es = 4 if dtype == "f32" else 8
        batch = _log_int(rng, 4, 256) if api == "batched" else 1
        m, n = _log_int(rng, 200, 100000), _log_int(rng, 200, 50000)
        if api == "centered" and m < 2 * n:
            continue
        k, p = _log_int(rng, 6, 512), rng.choice([4, 6, 8, 10, 10, 16, 20, 32, 64])
        q = rng.choice([1, 1, 2, 2, 3])
        l = k + p
        if 3 * l > min(m, n) or (api == "batched" and l > 128):
            continue
        entries, flops = batch * m * n, (2 * q + 2) * 2.0 * batch * m * n * l
        if entries * es > 4.3e9 or flops > (4.9e12 if dtype == "f32" else 1.3e12) or batch * l * l * 8 > 2e9:
            continue
        if rng.random() < 0.5:            # half of the shapes are round, as matrices in memory often are
            m, n = max(16, m // 16 * 16), max(16, n // 16 * 16)
        rate = round(rng.uniform(1.5, 4.0) / l, 5)
        rank = l + l // 2
        noise = round(0.2 * math.exp(-rate * rank) / (math.sqrt(m) + math.sqrt(n)), 9)
        return _case(None, api, dtype, m, n, k, p, q, rng.choice(["S", "SV", "SUV", "SUV"]), "exp", rate, rank, noise,
                     batch=batch)


def _spectrum(c, device):
    i = torch.arange(c["rank"], dtype=torch.float64, device=device)
    return torch.exp(-c["rate"] * i) if c["law"] == "exp" else (1.0 + i) ** -c["rate"]


def _orthonormal(shape, gen, device):
    """A Gaussian factor made orthonormal (Cholesky, twice), fp64."""
    X = torch.randn(shape, dtype=torch.float64, device=device, generator=gen)
    eye = torch.eye(shape[1], dtype=torch.float64, device=device)
    for _ in range(2):
        L = torch.linalg.cholesky(X.T.contiguous() @ X)
        X = X @ torch.linalg.solve_triangular(L, eye, upper=False).T.contiguous()
    return X


def _matrix(c, seed, device):
    """A (batch, m, n), in the type of the case, and the leading k planted right vectors as rows (batch, k, n)."""
    dt = torch.float32 if c["dtype"] == "f32" else torch.float64
    gen = torch.Generator(device=device)
    gen.manual_seed(int(seed))
    r, s = c["rank"], _spectrum(c, device)
    A = torch.empty((c["batch"], c["m"], c["n"]), dtype=dt, device=device)
    ref = torch.empty((c["batch"], c["k"], c["n"]), dtype=dt, device=device)
    # the blocks of a batch share their factors: other rows and another spread in each
    U, V = _orthonormal((c["m"], r), gen, device), _orthonormal((c["n"], r), gen, device)
    Ut, Vt = (U * s).to(dt), V.T.to(dt).contiguous()
    for b in range(c["batch"]):
        torch.matmul(Ut if b == 0 else torch.roll(Ut, 17 * b, 0), Vt if b == 0 else torch.roll(Vt, 29 * b, 1), out=A[b])
        ref[b] = torch.roll(Vt[: c["k"]], 29 * b, 1)
        if c["noise"]:
            rows = max(1, (1 << 26) // c["n"])
            for i in range(0, c["m"], rows):
                A[b, i:i + rows].add_(torch.randn(A[b, i:i + rows].shape, dtype=dt, device=device, generator=gen),
                                      alpha=c["noise"])
    if c["api"] == "centered":
        A += torch.randn(c["n"], dtype=dt, device=device, generator=gen) * (2.0 / math.sqrt(c["m"]))
    return A, ref


def prepare(case, seed):
    A, ref = _matrix(case, seed, "cuda")
    if case["api"] != "batched":
        A, ref = A[0], ref[0]
    return {"case": case, "A": A, "ref": ref, "ctx": Rsvd(0)}


def run(state):
    c, ctx = state["case"], state["ctx"]
    args = dict(k=c["k"], p=c["p"], q=c["q"], seed=SKETCH_SEED, job=JOBS[c["job"]], want_info=c["info"])
    mean = None
    if c["api"] == "run":
        S, U, Vt, _ = ctx.rsvd_run(state["A"], **args)
    elif c["api"] == "centered":
        S, U, Vt, _, mean = ctx.rsvd_run_centered(state["A"], **args)
    else:
        S, U, Vt, _ = ctx.rsvd_run_batched(state["A"], **args)
    return _outputs(S, U, Vt, mean, state["ref"])


def _outputs(S, U, Vt, mean, ref):
    out = {"S": S}
    if Vt is not None:
        turn = torch.sign(torch.linalg.vecdot(Vt, ref))
        out["Vt"] = Vt.mul_(turn.unsqueeze(-1))
        if U is not None:
            out["U"] = U.mul_(turn.unsqueeze(-2))
    if mean is not None:
        out["mean"] = mean
    return out


def work(case):
    """Every entry of A in once and every output out once; the products with A (2q + 2 of them), a triangular
    factorisation of each of their results but the last, the factor of B and the outputs' products."""
    m, n, k, q, b = case["m"], case["n"], case["k"], case["q"], case["batch"]
    l, es = k + case["p"], 4 if case["dtype"] == "f32" else 8
    vt, u = case["job"] != "S", case["job"] == "SUV"
    values = m * n + k + (k * n if vt else 0) + (m * k if u else 0) + (n if case["api"] == "centered" else 0)
    flops = (2 * q + 2) * 2 * m * n * l + ((q + 1) * m + (q + 1) * n) * 2 * l * l
    flops += (2 * n * l * k if vt else 0) + (2 * m * l * k if u else 0)
    return {"bytes": float(b * values * es), "flops": float(b * flops)}


def tolerance(case):
    """A vector moves by about eps * s_j / (s_j - s_j+1) when sums are taken in another order.  Against `exact` the
    calls above show 2 to 7 times the root mean square of that in fp32 (up to 14 times in fp64: more products with A
    behind each other), values 5 eps (fp64: 50); allowed is four times as much."""
    f32 = case["dtype"] == "f32"
    eps = 2.0 ** -23 if f32 else 2.0 ** -52
    s = _spectrum(dict(case, rank=case["k"] + 1), "cpu")
    moved = float(torch.sqrt(torch.mean((eps * s[:-1] / (s[:-1] - s[1:])) ** 2))) if case["job"] != "S" else 0.0
    return {"rel": max((20.0 if f32 else 200.0) * eps, (25.0 if f32 else 50.0) * moved)}


# ---- the same result in 64 bits

def _gaussian(seed, rows, cols, f32, device):
    """The sketch: Philox4x32-10 (Salmon, Moraes, Dror, Shaw, SC'11) and Box-Muller, in the stream layout that the
    library documents."""
    per, mask = (4 if f32 else 2), 0xFFFFFFFF
    groups = (rows * cols + per - 1) // per
    g = torch.arange(groups, dtype=torch.int64, device=device)
    c0, c1, c2, c3 = g & mask, g >> 32, torch.zeros_like(g), torch.zeros_like(g)
    k0, k1 = seed & mask, (seed >> 32) & mask
    for _ in range(10):
        p0, p1 = c0 * 0xD2511F53, c2 * 0xCD9E8D57
        c0, c1, c2, c3 = ((p1 >> 32) & mask) ^ c1 ^ k0, p1 & mask, ((p0 >> 32) & mask) ^ c3 ^ k1, p0 & mask
        k0, k1 = (k0 + 0x9E3779B9) & mask, (k1 + 0xBB67AE85) & mask
    if f32:
        u = [((x >> 8).double() + 0.5) * 2.0 ** -24 for x in (c0, c1, c2, c3)]
    else:
        u = [(((hi << 20) | (lo >> 12)).double() + 0.5) * 2.0 ** -52 for hi, lo in ((c0, c1), (c2, c3))]
    z = []
    for a, b in zip(u[0::2], u[1::2]):
        r, t = torch.sqrt(-2.0 * torch.log(a)), (2.0 * math.pi) * b
        z += [r * torch.cos(t), r * torch.sin(t)]
    flat = torch.stack(z, dim=1).reshape(-1)[: rows * cols]
    return (flat.float().double() if f32 else flat).reshape(rows, cols)


def _basis(Y):
    return torch.linalg.qr(Y.cpu())[0].to(Y.device)


def _times(A, X, transpose=False):
    """A X or A^T X in fp64, a block of rows of A at a time."""
    m, n = A.shape
    out = torch.zeros((n if transpose else m, X.shape[1]), dtype=torch.float64, device=A.device)
    step = max(1, (1 << 27) // n)
    for i in range(0, m, step):
        blk = A[i:i + step].double()
        if transpose:
            out += blk.T.contiguous() @ X[i:i + step]
        else:
            out[i:i + step] = blk @ X
    return out


def exact(case, seed):
    A, ref = _matrix(case, seed, "cuda")
    parts = []
    for b in range(case["batch"]):
        parts.append(_exact_one(case, A[b], ref[b], SKETCH_SEED + b))
    if case["api"] == "batched":
        return {key: torch.stack([x[key] for x in parts]) for key in parts[0]}
    return parts[0]


def _exact_one(c, A, ref, seed):
    l, k = c["k"] + c["p"], c["k"]
    mean = None
    ax, atx = (lambda X: _times(A, X)), (lambda X: _times(A, X, True))
    if c["api"] == "centered":
        mean = _times(A, torch.ones((c["m"], 1), dtype=torch.float64, device=A.device), True)[:, 0] / c["m"]
        ax = lambda X: _times(A, X) - mean @ X                                  # noqa: E731
        atx = lambda X: _times(A, X, True) - torch.outer(mean, X.sum(0))        # noqa: E731
    Q = _basis(ax(_gaussian(seed, c["n"], l, c["dtype"] == "f32", A.device)))
    for _ in range(c["q"]):
        Q = _basis(ax(_basis(atx(Q))))
    Qb, R = torch.linalg.qr(atx(Q).cpu())
    X, S, Wt = (torch.from_numpy(x) for x in np.linalg.svd(R.numpy()))
    dev = A.device
    Vt = (Qb @ X[:, :k]).T.contiguous().to(dev) if c["job"] != "S" else None
    U = Q @ Wt[:k].T.contiguous().to(dev) if c["job"] == "SUV" else None
    return _outputs(S[:k], U, Vt, mean, ref.double())
