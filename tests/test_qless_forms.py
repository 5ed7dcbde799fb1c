"""Algorithm 6 on dense A: which calls go column by column and which in blocks.
The rule on the CPU at sizes timed in both forms, and the scores on both sides of
its lines.  Bars as for the other sizes: 1e-10 relative per score in FP64, 1e-4
in the FP32-level forms."""

import ctypes

import numpy as np
import pytest
import torch

from oracle import leverage as L
from paper_2105_11004_amd import api


@pytest.mark.parametrize("n,d,k,elt,blocks", [
    (1 << 20, 1, 1, 4, False), (1 << 20, 4, 4, 8, False), (1 << 20, 8, 8, 2, False), (1 << 20, 16, 4, 4, False),
    (1 << 20, 32, 4, 4, False), (1 << 20, 32, 4, 8, True), (131000, 32, 4, 8, False), (33000, 64, 2, 8, False),
    (33000, 16, 4, 4, False), (131000, 8, 8, 4, True), (60000, 4, 4, 4, True), (262000, 4, 4, 4, False),
    (9999, 16, 4, 4, True), (16000, 16, 4, 4, False),
    (1000, 1, 1, 4, True), (1 << 20, 64, 4, 4, True), (50000, 256, 1, 4, True), (1 << 20, 16, 16, 2, True),
    (1 << 20, 256, 16, 4, True), (1 << 20, 257, 1, 4, False)])
def test_qless_form_is_the_faster_one(n, d, k, elt, blocks):
    rule = getattr(api.load_library(), "_ZN3lev15qless_in_blocksEllll")
    rule.argtypes, rule.restype = [ctypes.c_int64] * 4, ctypes.c_bool
    assert rule(n, d, k, elt) is blocks


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,prec,bar", [(torch.float64, "native", 1e-10), (torch.float32, "native", 1e-4),
                                            (torch.bfloat16, "bf16x3", 1e-4)], ids=["f64", "f32", "bf16"])
@pytest.mark.parametrize("n,d,cap", [(9999, 16, 4), (10000, 16, 4), (10001, 64, 2), (10001, 65, 2), (20011, 33, 3),
                                     (140003, 32, 4), (65537, 7, 5), (400003, 8, 8), (400003, 1, 1)])
def test_qless_scores_beside_the_lines(gpu, dtype, prec, bar, n, d, cap):
    print("qless forms", dtype, n, d, cap, flush=True)
    rng = np.random.default_rng(1000 * d + cap)
    H = rng.integers(-8, 9, (n, d)).astype(np.float64) * 2.0 ** rng.integers(-2, 3, d)
    per = 16 // torch.tensor([], dtype=dtype).element_size()
    A = torch.full((n, (d + per - 1) // per * per + per), float("nan"), dtype=dtype, device=gpu)
    A[:, :d] = torch.from_numpy(H).to(dtype).to(gpu)
    theta = api.lev_estimate(A[:, :d], 0, 1, 1, cap, 1e-5, precision=prec, mode="qless")
    ref, q = L.ls_qless_qr(H, 1e-5, cap)
    assert q.rank == cap
    theta = theta.cpu().numpy().astype(np.float64)
    live = ref > 1e-12
    assert (np.abs(theta - ref)[live] / ref[live]).max() < bar
