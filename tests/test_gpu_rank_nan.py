"""A column holding a NaN is never a pivot, and R shows it at every width: its
entries are NaN in the rows of the rank, beside a factor of the other columns
that is as without it.  One size per form of the pivoted Cholesky (one wave,
one workgroup, panels in either LDS layout).  Bar: 1e-9 R_00 as in the other
tests of the factor."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("col", [0, 37])
@pytest.mark.parametrize("d,rank", [(64, 48), (64, 63), (200, 128), (300, 33), (300, 299), (700, 45), (700, 96)])
def test_nan_column_is_shown_and_never_a_pivot(gpu, d, rank, col):
    print("nan column", d, rank, col, flush=True)
    rng = np.random.default_rng(10 * d + rank)
    m, others = d + 40, np.delete(np.arange(d), col)
    At = rng.standard_normal((m, d))
    if rank < d - 1:
        At[:, others] = rng.standard_normal((m, rank)) @ rng.standard_normal((rank, d - 1))
    At[:, others] *= rng.uniform(0.5, 2.0, d - 1)
    o = L.qrcp_sign_normalised(At[:, others], 1e-5)
    assert o.rank == rank
    At[5, col] = np.nan
    perm, R, r = api.lev_rank_estimate(torch.from_numpy(At).to(gpu), 1e-5)
    perm, R = perm.cpu().numpy(), R.cpu().numpy()
    assert int(r.item()) == rank
    np.testing.assert_array_equal(perm[:rank], others[o.perm[:rank]])
    rest = np.setdiff1d(np.arange(d), perm[:rank])
    np.testing.assert_array_equal(perm[rank:], rest)
    want = np.full((rank, d), np.nan)
    want[:, others[o.perm]] = o.R[:rank]
    np.testing.assert_allclose(R[:rank], want[:, perm], atol=1e-9 * o.R[0, 0], rtol=0)  # (NaN where NaN)
    assert np.all(R[rank:] == 0)
