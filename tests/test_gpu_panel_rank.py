"""The panel form of the pivoted Cholesky (d > 256) at the edges of its panels,
of its waves and of the two LDS layouts (d <= 600 and beyond), full rank and
rank deficient with the rank inside, at the end of and past a half panel,
against DGEQP3 on the same sketch.  Bar as for the other sizes: 1e-9 R_00."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rank", [(257, 257), (288, 288), (301, 17), (384, 48), (385, 64), (512, 79), (599, 599),
                                    (600, 80), (601, 80), (602, 49), (640, 640), (897, 33), (1023, 96), (1024, 16)])
def test_panel_rank_estimate(gpu, d, rank):
    print("panel rank", d, rank, flush=True)
    rng = np.random.default_rng(100 * d + rank)
    m = d + 40
    At = rng.standard_normal((m, rank)) @ rng.standard_normal((rank, d)) if rank < d else rng.standard_normal((m, d))
    At *= rng.uniform(0.5, 2.0, d)
    perm, R, r = api.lev_rank_estimate(torch.from_numpy(At).to(gpu), 1e-5)
    o = L.qrcp_sign_normalised(At, 1e-5)
    assert int(r.item()) == o.rank == rank
    perm, R = perm.cpu().numpy(), R.cpu().numpy()
    np.testing.assert_array_equal(perm[:rank], o.perm[:rank])
    np.testing.assert_array_equal(perm[rank:], np.sort(o.perm[rank:]))
    want = np.empty((rank, d))
    want[:, o.perm] = o.R[:rank]
    np.testing.assert_allclose(R[:rank], want[:, perm], atol=1e-9 * o.R[0, 0], rtol=0)
    assert np.all(R[rank:] == 0)


def test_panel_exact_ties_take_the_lowest_column(gpu):
    """Orthogonal columns of equal norm: every step is a tie, across lanes and
    across waves."""
    for d in (300, 700):
        perm, R, r = api.lev_rank_estimate(2.0 * torch.eye(d, dtype=torch.float64, device=gpu), 1e-5)
        assert int(r.item()) == d
        np.testing.assert_array_equal(perm.cpu().numpy(), np.arange(d))
        np.testing.assert_array_equal(R.cpu().numpy(), 2.0 * np.eye(d))
