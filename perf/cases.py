"""Performance cases: the calls a user of the leverage-score library makes, at
the sizes the library is used at, with their inputs, their unavoidable work
and what they return in 64-bit arithmetic.

A case is a dict of plain values.  `call` says which path it takes:

  estimate  scores of a dense A through lev_estimate (one call with everything
            allocated, `keep` False) or through a kept EstimatePlan
  csr       the same for a CSR A
  train     scores with autograd, and the gradient of w^T theta (forward and
            backward)
  select    lev_sketch, then lev_rank_estimate: the rank-revealing column
            selection of Algorithm 4 by itself
  lstsq     lev_precondition, then lev_lsqr with that preconditioner

`mode`, `sketch` and `precision` are the library's own options.  Sizes are
the repository's workloads and test shapes, and the ranges around them.
"""

from __future__ import annotations

import math

import numpy as np
import torch

from paper_2105_11004_amd import api
from paper_2105_11004_amd import workloads

DEVICE = "cuda"
DTYPES = {"f64": torch.float64, "f32": torch.float32, "bf16": torch.bfloat16}
BYTES = {"f64": 8, "f32": 4, "bf16": 2}


def _case(call, n, d, dtype="f32", rank=0, r_cs=1024, m=0, k=48, zeta=1e-5, **more):
    """rank 0: full column rank."""
    c = dict(call=call, n=n, d=d, dtype=dtype, rank=rank, r_cs=r_cs, m=m or 2 * d, k=k, zeta=zeta, mode="jl",
             sketch="gauss", precision="native", keep=False)
    c.update(more)
    return c


def listed():
    return [
        # a small FP64 matrix at the FP64 rank cutoff: latency and launches
        _case("estimate", 4096, 64, "f64", r_cs=1024, m=256, k=32, zeta=1e-10, name="f64_4096x64"),
        # a small ragged FP32 matrix, one call with nothing kept
        _case("estimate", 8199, 64, "f32", rank=48, r_cs=1024, m=128, k=32, name="f32_8199x64"),
        # the ordinary size: a tall FP32 matrix of half its rank, coherent rows
        _case("estimate", 1 << 20, 256, "f32", rank=128, r_cs=4096, m=512, k=48, keep=True, name="f32_1Mx256"),
        # the largest: BF16 storage, FP32-level arithmetic, repeated calls
        _case("estimate", 1 << 22, 1024, "bf16", r_cs=16384, m=2048, k=64, zeta=1e-3, precision="bf16x3", keep=True,
              name="bf16_4Mx1024"),
        # the SRHT in place of the Gaussian stage, ragged sizes, two column tiles
        _case("estimate", 200003, 520, "bf16", r_cs=8192, m=1100, k=100, zeta=1e-3, precision="bf16x3", sketch="srht",
              name="bf16_srht_200003x520"),
        # exact scores of the selected columns (Algorithm 7)
        _case("estimate", 1 << 20, 256, "f32", rank=128, r_cs=4096, m=512, mode="exact", keep=True,
              name="f32_exact_1Mx256"),
        # Algorithm 6, no sketch, rank well below sqrt(d)
        _case("estimate", 1 << 20, 256, "f32", rank=16, r_cs=4096, m=512, k=32, mode="qless", keep=True,
              name="f32_qless_1Mx256"),
        # the largest sparse matrix: power-law rows, zero columns
        _case("csr", 1 << 23, 512, "f32", zero_cols=64, r_cs=8192, m=1024, k=64, keep=True, name="csr_8Mx512"),
        # exact scores of a sparse matrix
        _case("csr", 300007, 300, "f32", zero_cols=44, r_cs=4096, m=600, mode="exact", name="csr_exact_300007x300"),
        # scores inside a training step: forward and backward
        _case("train", 1 << 20, 256, "f32", rank=192, r_cs=4096, m=512, k=48, name="train_f32_1Mx256"),
        # column selection by itself, wide, at the FP64 cutoff
        _case("select", 100003, 600, "f64", rank=450, r_cs=4096, m=1200, zeta=1e-10, name="select_f64_100003x600"),
        # Section 6: an ill-conditioned least-squares problem
        _case("lstsq", 50000, 60, "f64", r_cs=18000, m=120, zeta=1e-10, method="svd", kappa=1e3, iters=40,
              name="lstsq_f64_50000x60"),
    ]


def _log_int(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    """One more case of the listed ranges: the sizes log-uniform, most of them
    odd; the storage type, rank, sketch, mode and precision at random."""
    call = rng.choice(["estimate", "estimate", "estimate", "estimate", "csr", "csr", "train", "train", "select",
                       "lstsq"])
    if call == "estimate":
        mode = rng.choice(["jl", "jl", "jl", "exact", "nojl", "qless"])
        d = _log_int(rng, 16, 256 if mode == "qless" else 1024)
        n = _log_int(rng, max(2000, 8 * d), max(16 * d, min(1 << 21, (1 << (28 if mode == "jl" else 26)) // d)))
        dtype = rng.choice(["f64", "f32", "f32", "bf16"]) if mode != "qless" else rng.choice(["f64", "f32"])
        if mode == "qless":
            rank = rng.randint(3, min(24, d // 2))
            return _case(call, n, d, dtype, rank=rank, k=rank + 8, mode=mode, keep=True)
        sketch = rng.choice(["gauss", "gauss", "gauss", "srht"])
        r_cs = _log_int(rng, 3 * d, 16 * d)
        if sketch == "srht":
            r_cs = 1 << r_cs.bit_length()
        rank = 0 if dtype == "bf16" or rng.random() < 0.5 else max(4, int(d * rng.uniform(0.3, 0.9)))
        return _case(call, n, d, dtype, rank=rank, r_cs=max(256, r_cs), m=int(d * rng.uniform(1.5, 2.5)) + 8,
                     k=rng.choice([16, 32, 48, 64, rng.randint(8, 160)]), mode=mode, sketch=sketch,
                     zeta={"f64": 1e-10, "f32": 1e-5, "bf16": 1e-3}[dtype],
                     precision=rng.choice(["native", "bf16x3"]) if dtype == "bf16" else "native",
                     keep=rng.random() < 0.5)
    if call == "csr":
        mode = rng.choice(["jl", "jl", "jl", "exact", "nojl"])
        d = _log_int(rng, 40, 768)
        n = _log_int(rng, max(20000, 24 * d), 1 << (21 if mode == "jl" else 19))
        dtype = rng.choice(["f64", "f32", "f32", "bf16"])
        return _case(call, n, d, dtype, zero_cols=d // 8, r_cs=_log_int(rng, 4 * d, 16 * d), m=2 * d,
                     k=rng.randint(8, 64), mode=mode, zeta=1e-10 if dtype == "f64" else 1e-5, keep=rng.random() < 0.5)
    if call == "train":
        d = rng.choice([16 * rng.randint(1, 16), _log_int(rng, 16, 320)])
        n = _log_int(rng, max(2000, 8 * d), (1 << 27) // d)
        return _case(call, n, d, rng.choice(["f32", "f32", "f64"]), rank=rng.choice([0, max(4, 3 * d // 4)]),
                     r_cs=_log_int(rng, 4 * d, 16 * d), m=2 * d, k=rng.randint(8, 64), zeta=1e-5)
    if call == "select":
        d = _log_int(rng, 24, 1024)
        n = _log_int(rng, max(2000, 8 * d), (1 << 26) // d)
        return _case(call, n, d, "f64", rank=rng.choice([0, max(4, 3 * d // 4)]), r_cs=_log_int(rng, 3 * d, 12 * d),
                     m=2 * d, zeta=rng.choice([1e-10, 1e-5]))
    d = _log_int(rng, 16, 128)
    n = _log_int(rng, 10000, 1 << 19)
    return _case("lstsq", n, d, rng.choice(["f64", "f64", "f32"]), r_cs=5 * d * (d + 1) if d < 64 else 64 * d, m=2 * d,
                 zeta=1e-10, method=rng.choice(["svd", "qr"]), kappa=10.0 ** rng.randint(1, 3), iters=rng.randint(20, 60))


# ---------------------------------------------------------------- inputs
def _padded(A):
    """A with its rows padded to 16 bytes, which the library asks for."""
    n, d = A.shape
    per = 16 // A.element_size()
    if d % per == 0:
        return A
    B = torch.zeros(n, (d + per - 1) // per * per, dtype=A.dtype, device=A.device)
    B[:, :d] = A
    return B[:, :d]


def _matrix(c, seed):
    n, d, dtype = c["n"], c["d"], DTYPES[c["dtype"]]
    if c["call"] == "csr":
        return workloads.sparse_power_law(n, d, c["zero_cols"], seed, mean_nnz=min(16.0, d / 4), dtype=dtype,
                                          device=DEVICE, chunk=max(1 << 12, (1 << 25) // d))
    if c["call"] == "lstsq":
        sigma = torch.linspace(1.0, 1.0 / c["kappa"], d, dtype=torch.float64)
        return _padded(workloads.fixed_spectrum(n, sigma, seed, dtype=dtype, device=DEVICE))
    if c["dtype"] == "bf16":
        return _padded(workloads.row_scaled_bf16(n, d, seed, device=DEVICE))
    # a training step's matrix has no planted heavy rows
    heavy = 0.0 if c["call"] == "train" else 0.01
    if c["rank"]:
        return _padded(workloads.low_rank_coherent(n, d, c["rank"], seed, heavy_frac=heavy, dtype=dtype, device=DEVICE))
    return _padded(workloads.dense_gaussian(n, d, seed, dtype=dtype, device=DEVICE))


def _vector(c, seed):
    """w ~ U(0, 1) of a training step, b ~ N(0, 1) of a least-squares problem."""
    g = torch.Generator(device=DEVICE).manual_seed(seed + 1)
    if c["call"] == "train":
        return torch.rand(c["n"], generator=g, dtype=DTYPES[c["dtype"]], device=DEVICE)
    return torch.randn(c["n"], generator=g, dtype=torch.float64, device=DEVICE)


def prepare(case, seed):
    c = dict(case)
    A = _matrix(c, seed)
    s = {"c": c, "A": A, "seed": 2000 + seed}
    if c["call"] in ("train", "lstsq"):
        s["v"] = _vector(c, seed)
    if c["call"] == "train":
        A.requires_grad_(True)
    if c["keep"]:
        s["plan"] = api.EstimatePlan(A, s["seed"], c["r_cs"], c["m"], c["k"], c["zeta"], precision=c["precision"],
                                     mode=c["mode"], sketch=c["sketch"])
    return s


def run(s):
    c, A = s["c"], s["A"]
    if c["call"] == "select":
        At = api.lev_sketch(A, s["seed"], c["r_cs"], c["m"])
        perm, R, rank = api.lev_rank_estimate(At, c["zeta"])
        return {"At": At, "perm": perm, "R": R, "rank": rank}
    if c["call"] == "lstsq":
        N, k = api.lev_precondition(A, s["seed"], c["r_cs"], c["m"], c["zeta"], method=c["method"])
        x, hist = api.lev_lsqr(A, N, s["v"], c["iters"])
        return {"N": N, "k": k, "x": x, "resid": hist}
    if c["call"] == "train":
        theta = api.estimate(A, s["seed"], c["r_cs"], c["m"], c["k"], c["zeta"])
        (g,) = torch.autograd.grad(theta, A, grad_outputs=s["v"])
        return {"theta": theta.detach(), "grad": g}
    if c["keep"]:
        return {"theta": s["plan"].run()}
    if c["mode"] == "jl":
        theta, state = api.lev_estimate(A, s["seed"], c["r_cs"], c["m"], c["k"], c["zeta"], precision=c["precision"],
                                        return_state=True, sketch=c["sketch"])
        return {"theta": theta, "rank": state.rank}
    return {"theta": api.lev_estimate(A, s["seed"], c["r_cs"], c["m"], c["k"], c["zeta"], precision=c["precision"],
                                      mode=c["mode"], sketch=c["sketch"])}


def work(case):
    """A read once and the outputs written once; the operations of the steps
    at the case's rank.  A sparse matrix has its mean of nonzeros in a row."""
    c = case
    n, d, m, r_cs, b = c["n"], c["d"], c["m"], c["r_cs"], BYTES[c["dtype"]]
    nnz_row = min(16.0, d / 4) if c["call"] == "csr" else float(d)
    r = c["rank"] or (d - c["zero_cols"] if c["call"] == "csr" else d)
    a_bytes = n * nnz_row * (b + 4) + 8 * n if c["call"] == "csr" else n * d * b
    out = n * (8 if c["dtype"] == "f64" else 4)
    stage = 2.0 * m * r_cs * d if c["sketch"] == "gauss" else r_cs * d * math.log2(r_cs)
    sketch = n * nnz_row + stage + m * d * d
    if c["call"] == "select":
        return {"bytes": a_bytes + 8.0 * (m * d + d * d), "flops": sketch + r * r * d}
    if c["call"] == "lstsq":
        return {"bytes": a_bytes + 8.0 * (n + d * d), "flops": sketch + c["iters"] * 4.0 * n * d}
    if c["mode"] == "qless":
        return {"bytes": a_bytes + out, "flops": 2.0 * n * d * r + 2.0 * n * r * r}
    cols = c["k"] if c["mode"] == "jl" else r
    flops = sketch + r * r * d + 2.0 * n * nnz_row * cols
    if c["mode"] == "exact":
        flops += n * nnz_row * nnz_row
    if c["call"] == "train":
        return {"bytes": 2.0 * a_bytes + 2 * out, "flops": flops + 6.0 * n * d * cols + 2.0 * m * r_cs * d}
    return {"bytes": a_bytes + out, "flops": flops}


# ---------------------------------------------------------------- 64 bits
# What the calls return, by definition, in FP64 torch and numpy.  The random
# objects are defined by published generators, so they are written out here.
MASK32 = (1 << 32) - 1
MASK64 = (1 << 64) - 1
P61 = (1 << 61) - 1
GAMMA = 0x9E3779B97F4A7C15


def _mix64(z):
    """SplitMix64's output function on a uint64 array."""
    z = np.asarray(z, dtype=np.uint64)
    z = (z ^ (z >> np.uint64(30))) * np.uint64(0xBF58476D1CE4E5B9)
    z = (z ^ (z >> np.uint64(27))) * np.uint64(0x94D049BB133111EB)
    return z ^ (z >> np.uint64(31))


def _words(seed):
    return [int(w) for w in _mix64(np.array([(seed + (t + 1) * GAMMA) & MASK64 for t in range(10)], dtype=np.uint64))]


def _prime_from(x):
    while any(x % f == 0 for f in range(2, math.isqrt(x) + 1)):
        x += 1
    return x


def _hash(seed, n, r_cs):
    """Bucket and sign of every row: ((a i + c) mod P) mod r_cs, and the parity
    of a cubic over GF(2^61 - 1)."""
    w, P = _words(seed), _prime_from(max(n, 2))
    i = np.arange(n, dtype=np.uint64)
    h = (np.uint64(1 + w[0] % (P - 1)) * i + np.uint64(w[1] % P)) % np.uint64(P) % np.uint64(r_cs)
    g = np.full(n, w[5] % P61, dtype=np.uint64)
    p, low = np.uint64(P61), np.uint64((1 << 29) - 1)
    for t in (2, 1, 0):  # Horner; g = hi 2^32 + lo, and 2^61 = 1
        hi, lo = (g >> np.uint64(32)) * i, (g & np.uint64(MASK32)) * i
        g = ((hi >> np.uint64(29)) + ((hi & low) << np.uint64(32))) % p + ((lo & p) + (lo >> np.uint64(61))) % p
        g = (g % p + np.uint64(w[2 + t] % P61)) % p
    sign = 1.0 - 2.0 * (g & np.uint64(1)).astype(np.float64)
    return torch.from_numpy(h.astype(np.int64)).to(DEVICE), torch.from_numpy(sign).to(DEVICE)


def _gaussian(key, rows, cols):
    """rows x cols N(0, 1) / sqrt(rows): Philox4x32-10, Box-Muller on pairs of
    consecutive row-major elements."""
    pairs = (rows * cols + 1) // 2
    x0 = torch.arange(pairs, dtype=torch.int64, device=DEVICE)
    x1, x2, x3 = x0 >> 32, torch.zeros_like(x0), torch.zeros_like(x0)
    x0 = x0 & MASK32
    k0, k1 = key & MASK32, key >> 32
    for _ in range(10):
        p0, p1 = x0 * 0xD2511F53, x2 * 0xCD9E8D57  # the low 64 bits, as signed words
        x0, x1, x2, x3 = ((p1 >> 32) & MASK32) ^ x1 ^ k0, p1 & MASK32, ((p0 >> 32) & MASK32) ^ x3 ^ k1, p0 & MASK32
        k0, k1 = (k0 + 0x9E3779B9) & MASK32, (k1 + 0xBB67AE85) & MASK32
    u1 = (((x0 << 21) | (x1 >> 11)).double() + 0.5) * 2.0 ** -53
    u2 = (((x2 << 21) | (x3 >> 11)).double() + 0.5) * 2.0 ** -53
    radius, angle = torch.sqrt(-2.0 * torch.log(u1)), 2.0 * math.pi * u2
    return torch.stack([radius * torch.cos(angle), radius * torch.sin(angle)], 1).reshape(-1)[:rows * cols].reshape(rows, cols)


def _srht(w, X, m):
    """P H D X / sqrt(m): signs, the Walsh-Hadamard butterflies, and the first
    m coordinates of a four-round Feistel permutation walked into range."""
    r, d = X.shape
    gamma = np.uint64(GAMMA)
    D = 1.0 - 2.0 * (_mix64(np.uint64(w[8]) + np.arange(r, dtype=np.uint64) * gamma) >> np.uint64(63)).astype(np.float64)
    Y, step = X * torch.from_numpy(D).to(DEVICE)[:, None], 1
    while step < r:
        Y = Y.reshape(r // (2 * step), 2, step, d)
        Y = torch.stack([Y[:, 0] + Y[:, 1], Y[:, 0] - Y[:, 1]], 1).reshape(r, d)
        step *= 2
    half = max(1, ((r - 1).bit_length() + 1) // 2)
    mask = np.uint64((1 << half) - 1)
    at, todo = np.arange(m, dtype=np.uint64), np.ones(m, dtype=bool)
    while todo.any():
        left, right = at[todo] >> np.uint64(half), at[todo] & mask
        for t in range(4):
            f = _mix64(np.uint64(w[9]) + (np.uint64(t << 32) + right) * gamma) & mask
            left, right = right, left ^ f
        at[todo] = (left << np.uint64(half)) | right
        todo = at >= r
    return Y[torch.from_numpy(at.astype(np.int64)).to(DEVICE)] / math.sqrt(m)


def _blocks(c, A):
    """(first row, FP64 rows) of A in order, dense."""
    n, d = c["n"], c["d"]
    step = max(1, (1 << 27) // d)
    for lo in range(0, n, step):
        hi = min(n, lo + step)
        if c["call"] == "csr":
            ptr = A.row_ptr[lo:hi + 1]
            at = slice(int(ptr[0]), int(ptr[-1]))
            rows = torch.repeat_interleave(torch.arange(hi - lo, device=DEVICE), ptr[1:] - ptr[:-1])
            B = torch.zeros(hi - lo, d, dtype=torch.float64, device=DEVICE)
            B[rows, A.col_idx[at].long()] = A.values[at].double()
            yield lo, B
        else:
            yield lo, A[lo:hi].double()


def _sketch(c, A, seed):
    h, sign = _hash(seed, c["n"], c["r_cs"])
    SA = torch.zeros(c["r_cs"], c["d"], dtype=torch.float64, device=DEVICE)
    for lo, B in _blocks(c, A):
        SA.index_add_(0, h[lo:lo + len(B)], B * sign[lo:lo + len(B), None])
    w = _words(seed)
    return _srht(w, SA, c["m"]) if c["sketch"] == "srht" else _gaussian(w[6], c["m"], c["r_cs"]) @ SA / math.sqrt(c["m"])


def _pivoted_qr(At, zeta):
    """Column-pivoted Gram-Schmidt, each new direction orthogonalised again:
    the pivots in order and the rows of R (unpermuted columns)."""
    W, d = At.clone(), At.shape[1]
    Q = torch.zeros(At.shape[0], d, dtype=torch.float64, device=DEVICE)
    R = torch.zeros(d, d, dtype=torch.float64, device=DEVICE)
    perm, first = [], 0.0
    for j in range(d):
        norms = W.square().sum(0)
        norms[perm] = -1.0
        p = int(torch.argmax(norms))
        size = math.sqrt(max(float(norms[p]), 0.0))
        first = first or size
        if size <= zeta * first:
            break
        q = W[:, p]
        for _ in range(2):
            q = q - Q[:, :j] @ (Q[:, :j].T @ q)
        q = q / torch.linalg.norm(q)
        row = q @ W
        row[perm] = 0.0
        W -= torch.outer(q, row)
        Q[:, j], R[j] = q, row
        perm.append(p)
    return perm, R[:len(perm)]


def _pivoted_gram(B, zeta, cap):
    """Algorithm 6's recurrences on B = A^T A: the pivots and R."""
    norms, perm = torch.diagonal(B).clone(), []
    R = torch.zeros(0, B.shape[0], dtype=torch.float64, device=DEVICE)
    first = 0.0
    while len(perm) < min(cap, B.shape[0]):
        left = norms.clone()
        left[perm] = -1.0
        p = int(torch.argmax(left))
        size = math.sqrt(max(float(left[p]), 0.0))
        first = first or size
        if size <= zeta * first:
            break
        row = (B[p] - R[:, p] @ R) / size
        row[perm] = 0.0
        row[p] = size
        norms -= row.square()
        R = torch.cat([R, row[None]])
        perm.append(p)
    return perm, R


def _gram(c, A):
    B = torch.zeros(c["d"], c["d"], dtype=torch.float64, device=DEVICE)
    for _, X in _blocks(c, A):
        B += X.T @ X
    return B


def _scores(c, A, perm, X):
    """||e_i^T A_K X||^2, in the type the call returns, before its rounding."""
    return torch.cat([(B[:, perm] @ X).square().sum(1) for _, B in _blocks(c, A)])


def _solve(R, B):
    return torch.linalg.solve_triangular(R, B, upper=True)


def _lsqr(A, N, b, iters):
    """LSQR (Paige and Saunders) on A N from zero: x = N y and the residual
    norm after each step."""
    beta = torch.linalg.norm(b)
    u = b / beta
    v = N.T @ (A.T @ u)
    alpha = torch.linalg.norm(v)
    v = v / alpha
    w, y, phibar, rhobar, hist = v.clone(), torch.zeros_like(v), beta, alpha, []
    for _ in range(iters):
        u = A @ (N @ v) - alpha * u
        beta = torch.linalg.norm(u)
        u = u / beta
        v = N.T @ (A.T @ u) - beta * v
        alpha = torch.linalg.norm(v)
        v = v / alpha
        rho = torch.hypot(rhobar, beta)
        cos, sin = rhobar / rho, beta / rho
        theta, rhobar, phi, phibar = sin * alpha, -cos * alpha, cos * phibar, sin * phibar
        y, w = y + (phi / rho) * w, v - (theta / rho) * w
        hist.append(phibar)
    return N @ y, torch.stack(hist)


def exact(case, seed):
    c, sketch_seed = dict(case), 2000 + seed
    A = _matrix(c, seed)
    if c["mode"] == "qless":
        perm, R = _pivoted_gram(_gram(c, A), c["zeta"], c["k"])
        return {"theta": _scores(c, A, perm, torch.linalg.inv(R[:, perm]))}
    At = _sketch(c, A, sketch_seed)
    if c["call"] == "lstsq":
        _, sv, Vt = torch.linalg.svd(At, full_matrices=False)
        x, hist = _lsqr(A.double(), Vt.T / sv, _vector(c, seed), c["iters"])
        return {"N": None, "k": None, "x": x, "resid": hist}  # N: up to signs and rotations
    perm, R = _pivoted_qr(At, c["zeta"])
    r = len(perm)
    R11 = R[:, perm]
    if c["call"] == "select":
        rest = [j for j in range(c["d"]) if j not in set(perm)]
        full = torch.zeros(c["d"], c["d"], dtype=torch.float64, device=DEVICE)
        full[:r] = torch.cat([torch.triu(R11), R[:, rest]], 1)
        return {"At": At, "perm": None, "R": full, "rank": None}
    if c["mode"] == "exact":
        # A_K = Q R_B with R_B from the Gram of A_K R11^{-1}, which is well conditioned
        T = torch.linalg.inv(R11)
        B = torch.zeros(r, r, dtype=torch.float64, device=DEVICE)
        for _, X in _blocks(c, A):
            Y = X[:, perm] @ T
            B += Y.T @ Y
        theta = _scores(c, A, perm, T @ torch.linalg.inv(torch.linalg.cholesky(B).T))
    elif c["mode"] == "nojl":
        theta = _scores(c, A, perm, torch.linalg.inv(R11))
    else:
        Z = _solve(R11, _gaussian(_words(sketch_seed)[7], c["d"], c["k"])[:r] / math.sqrt(c["k"]))
        theta = _scores(c, A, perm, Z)
    if c["call"] != "train":
        return {"theta": theta, "rank": None} if c["mode"] == "jl" and not c["keep"] else {"theta": theta}
    # the adjoint at a fixed sketch, pivots and rank
    h, sign = _hash(sketch_seed, c["n"], c["r_cs"])
    w2 = 2.0 * _vector(c, seed).double()[:, None]
    AK = A.double()[:, perm]
    Y = w2 * (AK @ Z)
    Q = _solve(R11.T.flip(0, 1), At[:, perm].T.flip(0)).flip(0).T  # A~_K R11^{-1}, R11^T lower
    Rbar = -torch.triu(torch.linalg.solve_triangular(R11.T, (AK.T @ Y) @ Z.T, upper=False))
    M = R11 @ Rbar.T
    M = torch.tril(M) + torch.tril(M, -1).T
    H = _solve(R11, (Q @ M).T).T
    H = _gaussian(_words(sketch_seed)[6], c["m"], c["r_cs"]).T @ H / math.sqrt(c["m"])
    grad = torch.zeros(c["n"], c["d"], dtype=torch.float64, device=DEVICE)
    grad[:, perm] = Y @ Z.T + sign[:, None] * H[h]
    return {"theta": theta, "grad": grad}
