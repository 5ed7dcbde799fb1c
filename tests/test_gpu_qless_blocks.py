"""Algorithm 6 on dense A with d <= 256: rows of the Gram formed for blocks of
16 columns a pass.  Edges of the column blocks, step caps around one block,
more pivots than one block gives, and few rows; the rows' padding is NaN.
Bars as for the other sizes: 1e-10 relative per score in FP64, 1e-4 in the
FP32-level forms."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype,prec,bar", [(torch.float64, "native", 1e-10), (torch.float32, "native", 1e-4),
                                            (torch.bfloat16, "bf16x3", 1e-4)], ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,d,cap", [(1, 1, 1), (40, 17, 17), (3001, 16, 15), (5003, 63, 16), (5003, 64, 64),
                                     (4099, 65, 17), (6001, 128, 40), (6001, 129, 33), (7001, 192, 48),
                                     (7001, 193, 20), (70001, 256, 24)])
def test_qless_column_blocks(gpu, dtype, prec, bar, n, d, cap):
    print("qless blocks", dtype, n, d, cap, flush=True)
    rng = np.random.default_rng(1000 * d + cap)
    # powers of two spread over the columns: the pivots are not all among the
    # first block's columns, and A is exact in every type
    H = rng.integers(-8, 9, (n, d)).astype(np.float64) * 2.0 ** rng.integers(-2, 3, d)
    H[:, 0] += 1.0
    per = 16 // torch.tensor([], dtype=dtype).element_size()
    A = torch.full((n, (d + per - 1) // per * per + per), float("nan"), dtype=dtype, device=gpu)
    A[:, :d] = torch.from_numpy(H).to(dtype).to(gpu)
    A = A[:, :d]
    host = A.cpu().to(torch.float64).numpy()
    theta = api.lev_estimate(A, 0, 1, 1, cap, 1e-5, precision=prec, mode="qless").cpu().numpy().astype(np.float64)
    ref, q = L.ls_qless_qr(host, 1e-5, cap)
    assert abs(theta.sum() - q.rank) < 1e-3 * max(q.rank, 1)
    live = ref > 1e-12
    assert (np.abs(theta - ref)[live] / ref[live]).max() < bar
