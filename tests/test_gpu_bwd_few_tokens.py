"""Both gradients of a layer for few tokens on the vector kernels as one launch (dd_bwd), against the CPU oracle and, bit for
bit, against the two calls."""
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


# one token, remainders of groups and tiles, the last number of tokens it is made for and the next; diagonals shared between
# waves, more workgroups than one per diagonal, long sides either way
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", [(1, 1, 1, 1), (64, 64, 8, 16), (65, 63, 60, 3), (63, 257, 20, 15), (300, 100, 120, 33), (257, 255, 40, 192),
                                     (257, 255, 40, 193), (1001, 77, 300, 9), (100, 1030, 31, 130), (1200, 1100, 500, 41)])
def test_both_gradients(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + N + K + T)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    dX, dV = dd.dd_bwd(x, dy, off, V)
    assert rel_err(to_host(dX), orc.bwd_input(dY, offsets, values, M)) <= TOL[dtype]
    assert rel_err(to_host(dV), orc.bwd_weight(X, dY, offsets)) <= TOL_DV
    assert torch.equal(dX, dd.dd_bwd_input(dy, off, V, M)) and torch.equal(dV, dd.dd_bwd_weight(x, dy, off))
