"""The tile of the vector products: columns laid out once more behind the last one, zeros around a source narrower than the
destination.  Offsets that put the wrap at every place of a block of 64 columns, widths around 64, odd ones and odd addresses."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, random_case, rel_err, to_dev, to_host
from tests.test_gpu_vector import _by_diagonals

pytestmark = pytest.mark.gpu


# all diagonals: every offset, so every place of the wrap; both ways between sides that differ by less than, exactly and more than 64
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,T", [(1, 1, 3), (3, 2, 5), (7, 40, 33), (63, 63, 4), (64, 64, 33), (65, 65, 8), (64, 127, 9), (64, 128, 17),
                                   (66, 131, 9), (130, 194, 31), (130, 195, 12), (200, 199, 40)])
def test_every_offset(M, N, T, dtype):
    D = max(M, N)
    offsets, values, X, dY = random_case(M, N, D, T, dtype, seed=M + 3 * N + T)
    offsets = np.arange(D, dtype=np.int32)
    v = dd.DD_ALGO_VECTOR
    off, V = torch.from_numpy(offsets).cuda(), to_dev(values, dtype)
    for shift in (0, 1):  # rows on odd elements: no two columns to a load
        at = lambda a: torch.cat([to_dev(a, dtype).flatten()[:shift], to_dev(a, dtype).flatten()])[shift:].view(a.shape)
        assert rel_err(to_host(dd.dd_fwd(at(X), off, V, N, algo=v)), orc.fwd(X, offsets, values, N)) <= TOL[dtype]
        assert rel_err(to_host(dd.dd_bwd_input(at(dY), off, V, M, algo=v)), orc.bwd_input(dY, offsets, values, M)) <= TOL[dtype]


# the edges of a batch of eight diagonals, of 64 read at once and of 256 listed at once, by themselves
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("K", [1, 2, 7, 8, 9, 15, 16, 63, 64, 65, 71, 72, 255, 256, 257, 264, 265])
def test_numbers_of_diagonals(K, dtype):
    M, N, T = 290, 270, 600  # more tiles than a diagonal's parts would pay for
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=K)
    X[0, 0], dY[1, N - 1] = np.inf, -np.inf  # an odd last diagonal has no partner that it may meet
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    for got, ref in ((dd.dd_fwd(x, off, V, N, algo=dd.DD_ALGO_VECTOR), _by_diagonals(X, offsets, values, M, N, False)),
                     (dd.dd_bwd_input(dy, off, V, M, algo=dd.DD_ALGO_VECTOR), _by_diagonals(dY, offsets, values, M, N, True))):
        got, finite = to_host(got), np.isfinite(ref)
        assert (np.isfinite(got) == finite).all() and rel_err(got[finite], ref[finite]) <= TOL[dtype]
