"""Row lengths at the edges of the CSR passes' pieces (four entries a step, 16
and 64 a load, 64 rows a task, eight rows a group of pass 1), in shuffled
order, with row counts that leave the last task and the last groups ragged."""

import numpy as np
import pytest
import scipy.sparse as sp
import torch

from oracle import conventions as C
from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu

EDGES = [0, 1, 2, 3, 4, 5, 7, 8, 9, 12, 13, 15, 16, 17, 18, 31, 32, 33, 47, 48, 49, 62, 63, 64, 65, 67, 68, 127, 128,
         129, 191, 192, 193]


def _matrix(lengths, d, seed):
    rng = np.random.default_rng(seed)
    cols = [np.sort(rng.choice(d, size=min(ell, d), replace=False)) for ell in lengths]
    ptr = np.concatenate([[0], np.cumsum([len(c) for c in cols])]).astype(np.int64)
    idx = np.concatenate(cols + [np.zeros(0, dtype=np.int64)]).astype(np.int32)
    vals = np.round(rng.standard_normal(len(idx)) * 8) + 0.5  # exact in every storage type; none is zero
    return ptr, idx, vals


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16, torch.float64])
@pytest.mark.parametrize("kind,n,d", [("edges", 4001, 200), ("edges", 4097, 598), ("edges", 2999, 599), ("short", 4033, 64),
                                      ("long", 1030, 512), ("even", 4160, 24), ("one", 8200, 40)])
def test_csr_row_length_edges(gpu, dtype, kind, n, d):
    """S A has exact partial sums, so it is bit-exact; theta is compared with
    the FP64 oracle's at the storage type's rounding of the k-vector's sums
    (float32 sums of at most d terms: 1e-4 relative, as in the other sparse
    parity tests; 1e-9 in FP64)."""
    rng = np.random.default_rng(n + d)
    pool = {"edges": [e for e in EDGES if e <= d] + [d], "short": [0, 1, 2, 3], "long": [64, 65, 130, 300, 512],
            "even": [16], "one": [1] * 9 + [2]}[kind]
    lengths = rng.choice(pool, size=n)
    ptr, idx, vals = _matrix(lengths, d, n)
    A = api.Csr(torch.from_numpy(ptr).to(gpu), torch.from_numpy(idx).to(gpu), torch.from_numpy(vals).to(dtype).to(gpu), n, d)
    S = sp.csr_matrix((vals, idx, ptr), shape=(n, d))
    r_cs, m, k, zeta, seed = 2048, 2 * d + 16, 40, 1e-5, 11
    _, SA = api.lev_sketch(A, seed, r_cs, m, return_sa=True)
    np.testing.assert_array_equal(SA.cpu().numpy(), L.countsketch_apply(C.derive(seed, n, r_cs), S))
    theta = api.lev_estimate(A, seed, r_cs, m, k, zeta).cpu().numpy().astype(np.float64)
    o = L.ls_hrn_approx(S, seed, r_cs, m, k, zeta)
    rel = np.abs(theta - o.theta) / np.maximum(np.abs(o.theta), 1e-300)
    rel[o.theta == 0] = np.abs(theta[o.theta == 0])
    print(kind, dtype, n, d, "rank", o.rank, "max rel", rel.max(), flush=True)
    assert rel.max() <= (1e-9 if dtype == torch.float64 else 1e-4)


@pytest.mark.parametrize("dtype", [torch.float32, torch.float64])
@pytest.mark.parametrize("kind,n,d", [("edges", 4001, 200), ("edges", 2999, 300), ("short", 4033, 64), ("long", 1030, 512)])
def test_csr_gram_row_length_edges(gpu, dtype, kind, n, d):
    """The Gram of sparse rows through the exact scores: rows of one load (at
    most 64 entries), longer ones, runs past 64 entries in a 128-column block.
    Bars as for the exact scores of other sparse matrices."""
    rng = np.random.default_rng(n + d)
    pool = {"edges": [e for e in EDGES if e <= d] + [d], "short": [0, 1, 2, 3], "long": [64, 65, 130, 300, 512]}[kind]
    ptr, idx, vals = _matrix(rng.choice(pool, size=n), d, n)
    A = api.Csr(torch.from_numpy(ptr).to(gpu), torch.from_numpy(idx).to(gpu), torch.from_numpy(vals).to(dtype).to(gpu), n, d)
    S = sp.csr_matrix((vals, idx, ptr), shape=(n, d))
    zeta = 1e-10 if dtype == torch.float64 else 1e-5
    theta = api.lev_estimate(A, 12, 4096, 2 * d, 1, zeta, mode="exact").cpu().numpy().astype(np.float64)
    o = L.ls_hrn_exact(S, 12, 4096, 2 * d, zeta)
    live = o.theta > 0
    assert np.all(theta[~live] == 0)
    rel = np.abs(theta[live] - o.theta[live]) / o.theta[live]
    print(kind, dtype, n, d, "rank", o.rank, "exact max rel", rel.max(), flush=True)
    assert rel.max() < (1e-10 if dtype == torch.float64 else 1e-4)
