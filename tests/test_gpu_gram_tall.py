"""The Gram of a tall dense A (whole triangle per workgroup) through the exact
scores, at the edges of its column blocks and with ragged rows, padded
leading dimensions and row remainders.  Bars as for the exact scores at other
sizes: 1e-10 relative per score in FP64, 1e-4 in the FP32-level forms."""

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu

N = 65536 + 5  # the smallest row count with enough splits for the tall form, and a remainder


@pytest.mark.parametrize("dtype,prec,bar", [(torch.float64, "native", 1e-10), (torch.float32, "native", 1e-4),
                                            (torch.bfloat16, "bf16x3", 1e-4)], ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("d", [2, 16, 63, 64, 65, 128, 129, 192, 193, 250, 256])
def test_exact_scores_tall_gram(gpu, dtype, prec, bar, d):
    print("tall gram", dtype, d, flush=True)
    rng = np.random.default_rng(d)
    H = torch.from_numpy(rng.standard_normal((N, d)) * rng.uniform(0.5, 2.0, (N, 1))).to(dtype)
    per = 16 // H.element_size()
    A = torch.full((N, (d + per - 1) // per * per + per), float("nan"), dtype=dtype, device=gpu)
    A[:, :d] = H.to(gpu)
    theta = api.lev_estimate(A[:, :d], 77, 2048, 2 * d, 1, 1e-5, precision=prec, mode="exact")
    want, rank = L.theta_gram(H.to(torch.float64).numpy(), 1e-8)
    assert rank == d
    rel = np.abs(theta.cpu().numpy().astype(np.float64) - want) / want
    assert rel.max() < bar
