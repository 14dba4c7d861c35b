"""The selection where the number of candidates per thread changes and its first pass counts into copies, with scores whose first byte is
spread, shared by all, or undefined, against the CPU oracle."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("kind", ["normal", "one byte", "ties", "undefined"])
@pytest.mark.parametrize("B,D", [(1, 512), (2, 513), (1, 768), (1, 769), (3, 1025), (1, 1536), (1, 1537), (1, 2049), (1, 3072), (2, 3073), (1, 4097), (1, 8192),
                                 (1, 8193), (300, 700), (300, 1400)])
def test_selection(B, D, kind):
    rng = np.random.default_rng(B + D)
    scores = rng.standard_normal((B, D)).astype(np.float32)
    if kind == "one byte":
        scores = (1.0 + 0.5 * rng.random((B, D))).astype(np.float32)
    if kind == "ties":
        scores = np.round(scores)
    if kind == "undefined":
        scores[rng.random((B, D)) < 0.6] = np.nan
        scores[0, :3] = np.inf, -np.inf, -0.0
    d_scores = torch.from_numpy(scores).cuda()
    for K in (1, D // 10, D - 1, D):
        want = orc.select(scores, K)
        assert np.array_equal(dd.dd_select_diagonals(d_scores, K).cpu().numpy(), want)
        assert np.array_equal(dd.dd_select_soft(d_scores, K, 0.5)[0].cpu().numpy(), want)
