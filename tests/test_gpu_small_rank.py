"""The one-wave pivoted Cholesky (d <= 64) and the sizes around it, against
DGEQP3 on the same sketch.  Bar: the factor carries about u kappa^2 from the
Gram (kappa <= 1e3 here: 1e-10), so 1e-9 R_00 as for the wider sizes."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("zeta", [1e-5, 1e-10])
@pytest.mark.parametrize("d,rank", [(2, 1), (3, 3), (15, 15), (16, 7), (17, 17), (32, 32), (33, 20), (48, 48),
                                    (63, 49), (64, 64), (64, 16), (65, 65)])
def test_small_rank_estimate(gpu, d, rank, zeta):
    print("small rank", d, rank, zeta, flush=True)
    rng = np.random.default_rng(100 * d + rank)
    m = 2 * d + 3
    At = rng.standard_normal((m, rank)) @ rng.standard_normal((rank, d)) if rank < d else rng.standard_normal((m, d))
    perm, R, r = api.lev_rank_estimate(torch.from_numpy(At).to(gpu), zeta)
    o = L.qrcp_sign_normalised(At, zeta)
    assert int(r.item()) == o.rank == rank
    perm, R = perm.cpu().numpy(), R.cpu().numpy()
    np.testing.assert_array_equal(perm[:rank], o.perm[:rank])
    np.testing.assert_array_equal(perm[rank:], np.sort(o.perm[rank:]))
    np.testing.assert_allclose(R[:rank, :rank], o.R[:rank, :rank], atol=1e-9 * o.R[0, 0], rtol=0)
    want = np.empty((rank, d))
    want[:, o.perm] = o.R[:rank]
    np.testing.assert_allclose(R[:rank], want[:, perm], atol=1e-9 * o.R[0, 0], rtol=0)
    assert np.all(R[rank:] == 0)


def test_small_rank_exact_ties_take_the_lowest_column(gpu):
    """Orthogonal columns of equal norm: every step is a tie."""
    for d in (5, 64):
        At = np.zeros((d + 2, d))
        At[np.arange(d), np.arange(d)] = 2.0
        perm, R, r = api.lev_rank_estimate(torch.from_numpy(At).to(gpu), 1e-5)
        assert int(r.item()) == d
        np.testing.assert_array_equal(perm.cpu().numpy(), np.arange(d))
        np.testing.assert_array_equal(R.cpu().numpy(), 2.0 * np.eye(d))
