"""The FP64 products at the edges of their 64 x 64 x 32 tiles: sketches whose
rows and columns fall short of, fill and pass a tile, in both operand
orientations (A~ = G (S A) reads both along their rows, the Gram one operand
against them), one column (where both strides of A~ are 1) included."""

import numpy as np
import pytest
import torch

from oracle import conventions as C
from oracle import leverage as L
from paper_2105_11004_amd import api

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,r_cs,m", [(1, 40, 5), (1, 64, 64), (2, 33, 31), (63, 129, 96), (64, 128, 97), (65, 160, 128),
                                      (127, 257, 193), (129, 300, 257), (300, 640, 461)])
def test_products_at_tile_edges(gpu, d, r_cs, m):
    """A~ against the oracle's product (the bound of an FP64 sum of r_cs
    terms), then R^T R against the Gram of A~ at full rank: R comes from a
    Gram with sums of m terms and a Cholesky of d steps, each entry off by at
    most (m + d) eps times the columns' norms (1e-13 at these sizes)."""
    rng = np.random.default_rng(d + m)
    n = 4000
    ld = d + d % 2
    buf = torch.full((n, ld), float("nan"), dtype=torch.float64)  # the padding takes no part
    buf[:, :d] = torch.from_numpy(rng.standard_normal((n, d)))
    A = buf[:, :d].numpy().copy()
    At = api.lev_sketch(buf.to(gpu)[:, :d], 9, r_cs, m)
    rnd = C.derive(9, n, r_cs)
    G, SA = C.gaussian_transform(rnd, m), L.countsketch_apply(rnd, A)
    err = np.abs(At.cpu().numpy() - G @ SA)
    assert np.all(err <= 1e-13 * (np.abs(G) @ np.abs(SA)) + 1e-300)
    perm, R, rank = api.lev_rank_estimate(At, 1e-5)
    r = min(m, d)
    assert int(rank.item()) == r
    X = At.cpu().numpy()[:, perm.cpu().numpy()]
    R = R.cpu().numpy()
    Gram = X.T @ X
    nrm = np.sqrt(np.diag(Gram))
    assert np.all(np.abs(R.T @ R - Gram) <= 1e-12 * np.outer(nrm, nrm))
