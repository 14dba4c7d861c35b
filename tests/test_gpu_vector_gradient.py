"""The tiled weight gradient of the vector family: how a tile gets to LDS (one or two columns a load, more columns than are on their
way at once, rows that end inside a group), and the sum over few and many chunks, whole and ragged."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


# even widths (two columns of bf16 a load), odd ones, one odd; fewer columns than a wave has lanes, one more than a block of 64 and of
# 128; wide sides; tokens that end inside a group of 4 and of 8, fewer tokens than a chunk each; 5, 40 and 250 chunks, K * L even and odd
@pytest.mark.parametrize("M,N,K,T", [(130, 66, 21, 3001), (129, 65, 21, 3001), (129, 66, 21, 3003), (6, 40, 9, 6000), (5, 33, 7, 6005), (2, 2, 2, 9001),
                                     (1, 1, 1, 7000), (64, 192, 96, 1025), (65, 193, 97, 1030), (2050, 96, 60, 700), (1999, 97, 60, 701),
                                     (700, 4400, 40, 260), (320, 1000, 100, 333), (97, 101, 101, 8191)])
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_against_the_oracle(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + 3 * N + 5 * K + T)
    off, x, dy = torch.from_numpy(offsets).cuda(), to_dev(X, dtype), to_dev(dY, dtype)
    got = dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_VECTOR)
    assert rel_err(to_host(got), orc.bwd_weight(X, dY, offsets)) <= TOL_DV
    # matrices that start on an odd element, gradients that do: the other width of loads, the same sums
    odd = lambda a: torch.cat([a.new_zeros(1), a.flatten()])[1:].view(a.shape)
    out = odd(torch.empty_like(got))
    assert torch.equal(dd.dd_bwd_weight(odd(x), odd(dy), off, dValues=out, algo=dd.DD_ALGO_VECTOR), got)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_tokens_past_the_end_add_nothing(dtype):
    """Rows past the last token are read from it once more: an infinite one counts once, for its own diagonals."""
    M, N, K, T = 96, 160, 11, 1003
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=3)
    X[T - 1, 5] = np.inf
    off, x, dy = torch.from_numpy(offsets).cuda(), to_dev(X, dtype), to_dev(dY, dtype)
    got = to_host(dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_VECTOR))
    assert (np.isinf(got[:, 5])).all() and np.isfinite(np.delete(got, 5, axis=1)).all()
