"""Products from sources too wide for the tile to pay, on both sides of the rule: the untiled kernels against the oracle at few
and many tokens, both orientations, odd widths."""
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", [(9801, 301, 30, 1), (9801, 301, 30, 63), (301, 9801, 30, 5), (4501, 4500, 10, 2), (4499, 4500, 10, 2),
                                     (6001, 6000, 20, 3), (6000, 6001, 300, 3), (9999, 9998, 7, 2), (10300, 40, 3, 70000)])
def test_wide_sources(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + 7 * N + T)
    offsets[-1] += 3 * max(M, N)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    rows = slice(0, T) if T <= 100 else [0, 1, T // 2, 65534, 65535, 65536, T - 1]
    Y = dd.dd_fwd(x, off, V, N, algo=dd.DD_ALGO_VECTOR)[rows]
    dX = dd.dd_bwd_input(dy, off, V, M, algo=dd.DD_ALGO_VECTOR)[rows]
    assert rel_err(to_host(Y), orc.fwd(X[rows], offsets, values, N)) <= TOL[dtype]
    assert rel_err(to_host(dX), orc.bwd_input(dY[rows], offsets, values, M)) <= TOL[dtype]


def test_more_tiles_than_one_grid_holds():
    """1.08e9 tokens of a 2 -> 1 layer (13 GB): the tokens behind the 2^32nd thread are worked too."""
    T = (1 << 30) + 5000000
    X = torch.ones((T, 2), device="cuda")
    X[:, 1] = 3.0
    X[T - 1, 0], X[(1 << 30) + 1, 1] = 7.0, -2.0
    offsets, values = torch.tensor([1], dtype=torch.int32, device="cuda"), torch.tensor([[0.5]], device="cuda")
    Y = torch.full((T, 1), float("nan"), device="cuda")
    dd.dd_fwd(X, offsets, values, 1, Y=Y, algo=dd.DD_ALGO_VECTOR)
    assert (Y[:(1 << 30) + 1] == 1.5).all() and Y[(1 << 30) + 1, 0] == -1.0 and (Y[(1 << 30) + 2:] == 1.5).all()
    dX = X
    dd.dd_bwd_input(Y, offsets, values, 2, dX=dX, algo=dd.DD_ALGO_VECTOR)
    assert (dX[:, 0] == 0).all() and dX[(1 << 30) + 1, 1] == -0.5 and dX[T - 1, 1] == 0.75
