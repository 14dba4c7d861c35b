"""Selection and soft weights of many score vectors: on either side of the rules that choose the threads of a workgroup (256, 2048
and 4096 candidates, 256 vectors), bit for bit what one vector by itself gives."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [1, 64, 65, 128, 129, 255, 256, 257, 512, 513, 1024, 1025, 2048, 2049, 4096, 4097])
def test_batches_and_single_vectors_agree(D):
    rng = np.random.default_rng(D)
    batch = 300
    scores = rng.standard_normal((batch, D)).astype(np.float32)
    scores[1] = np.round(scores[1])
    scores[2, ::3] = np.nan
    K = max(1, D // 3)
    x, g = torch.from_numpy(scores).cuda(), torch.from_numpy(rng.standard_normal((batch, D)).astype(np.float32)).cuda()
    got = dd.dd_select_diagonals(x, K)
    np.testing.assert_array_equal(got.cpu().numpy(), orc.select(scores, K))
    both, weights = dd.dd_select_soft(x, K, 0.5)
    alpha, grad = dd.dd_soft_topk(x, K, 0.5), dd.dd_soft_topk_bwd(x, K, 0.5, g)
    assert torch.equal(both, got)
    same = lambda a, b: torch.equal(torch.nan_to_num(a, nan=-7.0), torch.nan_to_num(b, nan=-7.0))
    assert same(weights, alpha)
    for i in (0, 1, 2, 255, 256, batch - 1):
        one = x[i:i + 1].contiguous()
        assert torch.equal(dd.dd_select_diagonals(one, K), got[i:i + 1])
        assert same(dd.dd_soft_topk(one, K, 0.5), alpha[i:i + 1])
        assert same(dd.dd_select_soft(one, K, 0.5)[1], alpha[i:i + 1])
        assert same(dd.dd_soft_topk_bwd(one, K, 0.5, g[i:i + 1].contiguous()), grad[i:i + 1])
    p = torch.softmax(x.double() / 0.5, dim=-1)
    rows = [i for i in range(batch) if i != 2]
    assert (alpha[rows].double() - torch.clamp(K * p[rows], max=1.0)).abs().max() <= 4e-6
