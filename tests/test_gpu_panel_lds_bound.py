"""The panels on either side of the width up to which a column's whole panel
fits LDS (619 columns), against DGEQP3 on the same sketch.  Bar as for the
other sizes: 1e-9 R_00."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,rank", [(618, 80), (619, 49), (619, 619), (620, 49), (621, 64)])
def test_panels_where_lds_is_full(gpu, d, rank):
    print("panel lds bound", d, rank, flush=True)
    rng = np.random.default_rng(100 * d + rank)
    m = d + 40
    At = rng.standard_normal((m, rank)) @ rng.standard_normal((rank, d)) if rank < d else rng.standard_normal((m, d))
    At *= rng.uniform(0.5, 2.0, d)
    perm, R, r = api.lev_rank_estimate(torch.from_numpy(At).to(gpu), 1e-5)
    o = L.qrcp_sign_normalised(At, 1e-5)
    assert int(r.item()) == o.rank == rank
    perm, R = perm.cpu().numpy(), R.cpu().numpy()
    np.testing.assert_array_equal(perm[:rank], o.perm[:rank])
    want = np.empty((rank, d))
    want[:, o.perm] = o.R[:rank]
    np.testing.assert_allclose(R[:rank], want[:, perm], atol=1e-9 * o.R[0, 0], rtol=0)
    assert np.all(R[rank:] == 0)
