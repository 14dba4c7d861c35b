"""The weights and their derivative where the number of threads and of scores held per thread changes: against the CPU oracle, and bit for bit
the same for a vector alone and among many (another number of threads, one order of additions)."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from paper_2506_11449_amd import synth
from tests.parity_util import rel_err, to_host

pytestmark = pytest.mark.gpu

TOL = 1e-5  # fp32 exponentials and sums against the fp64 oracle, as max|gpu - ref| / max|ref|


@pytest.mark.parametrize("D", [1, 255, 256, 257, 513, 1024, 1025, 2048, 2049, 4096, 4097, 5120, 6144, 6145, 8192, 8193, 12288, 12289, 16384, 16385])
def test_weights_and_derivative(D):
    K = max(1, D // 10)
    scores, g = synth.draw_scores(1, D, seed=D), np.random.default_rng(D).standard_normal((1, D)).astype(np.float32)
    d_scores, d_g = torch.from_numpy(scores).cuda(), torch.from_numpy(g).cuda()
    weights, grad = dd.dd_soft_topk(d_scores, K, 0.7), dd.dd_soft_topk_bwd(d_scores, K, 0.7, d_g)
    assert rel_err(to_host(weights), orc.soft_topk(scores, K, 0.7)) <= TOL
    if D > 1:
        assert rel_err(to_host(grad), orc.soft_topk_bwd(scores, K, 0.7, g)) <= TOL
    both = dd.dd_select_soft(d_scores, K, 0.7)
    assert torch.equal(both[1], weights) and np.array_equal(both[0].cpu().numpy(), orc.select(scores, K))
    if D <= 4097:
        many = d_scores.expand(300, D).contiguous()
        assert torch.equal(dd.dd_soft_topk(many, K, 0.7)[299:], weights)
        assert torch.equal(dd.dd_soft_topk_bwd(many, K, 0.7, d_g.expand(300, D).contiguous())[299:], grad)
