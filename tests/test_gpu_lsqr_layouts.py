"""LSQR's column layouts: one, two, four or any number of 64-column blocks in
the product with A, one, two or four columns a lane in the one with A^T, and
the step's splits from 64 to 1024 columns, at the edges of each (d = 1, 64 /
65, 128 / 129, 256, 512 / 513, 1024), with row counts below one round of a
workgroup, at its edge and past it, against the FP64 oracle's recurrences."""

import numpy as np
import pytest
import torch

from oracle import precondition as P
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu

STEPS = 4


@pytest.mark.parametrize("dtype", [torch.float64, torch.float32, torch.bfloat16])
@pytest.mark.parametrize("n,d", [(1, 1), (129, 1), (31, 3), (1025, 63), (1026, 64), (2051, 65), (1300, 128), (2049, 129),
                                 (3001, 256), (4100, 512), (4203, 513), (8195, 1022), (8200, 1024)])
def test_lsqr_column_layouts(gpu, dtype, n, d):
    """A few steps on a well-conditioned Gaussian A with a dense, well-
    conditioned N.  A sum of n terms is off by at most n eps (2e-12 here) and
    a step passes an error on by at most kappa(A N)^2 < 1e2 of it in all four
    steps, so 1e-9 bounds both the iterate and the residuals."""
    rng = np.random.default_rng(1000 * n + d)
    es = torch.tensor([], dtype=dtype).element_size()
    ld = -(-d * es // 16) * 16 // es
    buf = torch.full((n, ld), float("nan"), dtype=dtype)  # the padding takes no part
    buf[:, :d] = torch.from_numpy(rng.standard_normal((n, d))).to(dtype)
    N = np.eye(d) + rng.standard_normal((d, d)) * (0.1 / np.sqrt(d))
    b = rng.standard_normal(n)
    steps = min(STEPS, d)  # (d steps reach the solution: nothing is left to compare after)
    x, hist = api.lev_lsqr(buf.to(gpu)[:, :d], torch.from_numpy(N).to(gpu), torch.from_numpy(b).to(gpu), steps)
    xo, ho = P.preconditioned_lsqr(buf[:, :d].to(torch.float64).numpy(), N, b, steps)
    rel = np.linalg.norm(x.cpu().numpy() - xo) / np.linalg.norm(xo)
    print(dtype, n, d, "lsqr vs oracle", rel, flush=True)
    assert rel <= 1e-9
    np.testing.assert_allclose(hist.cpu().numpy(), ho, rtol=1e-9, atol=1e-9 * np.linalg.norm(b))
