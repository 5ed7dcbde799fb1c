"""The general backward passes at the edges of their tiles: row tiles of 64, 32
and 16 rows with ragged ends, columns that leave the last 16-column block (and
the last 16-byte vector of a padded row) partly filled, one to four 16-column
blocks of the k-vectors, Z in LDS and read from memory.  Bars as for the other
gradients: the row's largest entry times 1e-9 in FP64, 1e-5 in FP32."""

import numpy as np
import pytest
import torch

from oracle import gradient as Gr
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,n,d,k", [(torch.float64, 1501, 17, 16), (torch.float64, 1600, 100, 33),
                                         (torch.float64, 2063, 143, 64), (torch.float64, 2100, 250, 60),
                                         (torch.float64, 2600, 300, 48), (torch.float32, 1537, 33, 17),
                                         (torch.float32, 2049, 143, 64), (torch.float32, 2500, 250, 49),
                                         (torch.float32, 2700, 321, 5)])
def test_general_backward_tiles(gpu, dtype, n, d, k):
    rng = np.random.default_rng(n + d + k)
    per = 16 // torch.tensor([], dtype=dtype).element_size()
    ld = -(-d // per) * per
    buf = torch.full((n, ld), float("nan"), dtype=dtype)  # the padding takes no part
    buf[:, :d] = torch.from_numpy(rng.standard_normal((n, d))).to(dtype)
    A = buf.to(gpu)[:, :d]
    w = torch.from_numpy(rng.uniform(0, 1, n)).to(dtype)
    r_cs, m, zeta = 4 * d + 32, 2 * d + 8, 1e-5
    theta, st = api.lev_estimate(A, 7, r_cs, m, k, zeta, return_state=True)
    g = api.lev_estimate_backward(A, st, w.to(gpu), 7, r_cs, m, k, zeta).cpu().to(torch.float64).numpy()
    ref = Gr.estimate_and_gradient(buf[:, :d].to(torch.float64).numpy(), 7, r_cs, m, k, zeta, w.to(torch.float64).numpy())
    assert int(st.rank.item()) == ref.rank == d
    np.testing.assert_array_equal(st.perm.cpu().numpy(), ref.perm)
    scale = np.abs(ref.grad).max(axis=1, keepdims=True)
    rel = (np.abs(g - ref.grad) / np.where(scale > 0, scale, 1.0)).max()
    print(dtype, n, d, k, "gradient row-rel err", rel, flush=True)
    assert rel < (1e-9 if dtype == torch.float64 else 1e-5)
