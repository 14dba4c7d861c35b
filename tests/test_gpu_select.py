"""The selection at the edges of its threads and slots (1024 threads, 1, 4, 16 or 64 candidates each), and the update of the
active set on either side of them, bit for bit against the oracle."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc

pytestmark = pytest.mark.gpu

EDGES = [1, 63, 64, 65, 1023, 1024, 1025, 2048, 4095, 4096, 4097, 16384, 16385, 30001, 65535, 65536]


@pytest.mark.parametrize("D", EDGES)
def test_selection_at_the_edges(D):
    rng = np.random.default_rng(D)
    scores = rng.standard_normal((3, D)).astype(np.float32)
    scores[1] = np.round(scores[1])                 # mostly ties
    scores[2, ::3] = np.nan
    scores[2, 1::3] = -np.inf
    for K in sorted({1, (D + 1) // 2, max(1, D - 1), D}):
        ref = orc.select(scores, K)
        got = dd.dd_select_diagonals(torch.from_numpy(scores).cuda(), K).cpu().numpy()
        np.testing.assert_array_equal(got, ref)
        soft, alpha = dd.dd_select_soft(torch.from_numpy(scores).cuda(), K, 0.5)
        np.testing.assert_array_equal(soft.cpu().numpy(), ref)


@pytest.mark.parametrize("D,K,n_drop", [(1023, 500, 500), (1024, 1000, 24), (1025, 3, 0), (4096, 409, 100), (4097, 409, 409),
                                        (16384, 1600, 500), (16385, 16000, 385), (65536, 65000, 300)])
def test_update_at_the_edges(D, K, n_drop):
    rng = np.random.default_rng(D + K)
    offsets = rng.permutation(D)[:K].astype(np.int32)
    magnitudes = rng.integers(0, 50, K).astype(np.float32)
    random = rng.random(D).astype(np.float32)
    new, source = dd.dd_diagheur_update(D, torch.from_numpy(offsets).cuda(), torch.from_numpy(magnitudes).cuda(),
                                        torch.from_numpy(random).cuda(), n_drop)
    ref_new, ref_source = orc.diagheur_update(D, offsets, magnitudes, random, n_drop)
    np.testing.assert_array_equal(new.cpu().numpy(), ref_new)
    np.testing.assert_array_equal(source.cpu().numpy(), ref_source)
