"""The tiled kernels of the vector family at the sizes where they can go wrong: edges of the token tiles, of the 64-column
blocks, of the blocks and passes of diagonals, layers at the limit of LDS, and inputs that are not finite."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

# (M, N, K, T)
EDGES = [
    (65, 63, 9, 31), (64, 65, 8, 32), (63, 127, 17, 33), (129, 64, 24, 1),     # column blocks, tiles of 4 ... 32 tokens
    (300, 290, 25, 5), (290, 300, 49, 17), (257, 257, 73, 64),                 # blocks of 8, 16 and 24 diagonals
    (400, 400, 255, 40), (400, 410, 256, 9), (410, 400, 257, 40),              # passes of 256 diagonals, parts of them
    (600, 40, 513, 70), (40, 600, 513, 70),                                    # most diagonals miss a block of columns
    (1024, 1000, 300, 16),                                                     # few tokens: waves share a column block
    (1990, 70, 30, 100), (70, 1990, 30, 100), (3000, 33, 20, 50),              # shallow tiles, wide sources
    (5000, 40, 30, 37), (40, 5000, 30, 37), (9000, 24, 12, 21), (24, 10300, 12, 21),  # the limits of LDS
    (96, 96, 20, 5000), (333, 160, 40, 4001),                                  # many chunks of tokens
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", EDGES)
def test_tiled_kernels_against_the_oracle(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + 7 * N + 31 * K + T)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    v = dd.DD_ALGO_VECTOR
    assert rel_err(to_host(dd.dd_fwd(x, off, V, N, algo=v)), orc.fwd(X, offsets, values, N)) <= TOL[dtype]
    assert rel_err(to_host(dd.dd_bwd_input(dy, off, V, M, algo=v)), orc.bwd_input(dY, offsets, values, M)) <= TOL[dtype]
    assert rel_err(to_host(dd.dd_bwd_weight(x, dy, off, algo=v)), orc.bwd_weight(X, dY, offsets)) <= TOL_DV


def _by_diagonals(A, offsets, values, M, N, transposed):
    """The product diagonal by diagonal in 64 bits: an entry meets only the stored weights."""
    D, L = max(M, N), min(M, N)
    p = np.arange(L)
    out = np.zeros((A.shape[0], M if transposed else N))
    with np.errstate(invalid="ignore", over="ignore"):
        for o, v in zip(offsets, values.astype(np.float64)):
            q = (p + o) % D
            rows, cols = (p, q) if M <= N else (q, p)
            src, dst = (cols, rows) if transposed else (rows, cols)
            out[:, dst] += A[:, src].astype(np.float64) * v
    return out


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", [(100, 100, 13, 37), (100, 260, 31, 37), (260, 100, 31, 37), (256, 270, 1, 3)])
def test_inputs_that_are_not_finite_reach_their_own_diagonals_only(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=5)
    for A in (X, dY):
        A[1, 0], A[T - 1, A.shape[1] - 1], A[0, A.shape[1] // 2] = np.inf, -np.inf, np.nan
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    v = dd.DD_ALGO_VECTOR
    for got, ref in ((dd.dd_fwd(x, off, V, N, algo=v), _by_diagonals(X, offsets, values, M, N, False)),
                     (dd.dd_bwd_input(dy, off, V, M, algo=v), _by_diagonals(dY, offsets, values, M, N, True))):
        got = to_host(got)
        finite = np.isfinite(ref)
        assert (np.isfinite(got) == finite).all()
        assert rel_err(got[finite], ref[finite]) <= TOL[dtype]
    dV = to_host(dd.dd_bwd_weight(x, dy, off, algo=v))
    p = np.arange(min(M, N))
    with np.errstate(invalid="ignore", over="ignore"):
        for k, o in enumerate(offsets):
            q = (p + o) % max(M, N)
            rows, cols = (p, q) if M <= N else (q, p)
            ref = (X[:, rows].astype(np.float64) * dY[:, cols]).sum(0)
            assert (np.isfinite(dV[k]) == np.isfinite(ref)).all()
