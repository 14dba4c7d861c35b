"""The matrix-core weight gradient where it cuts the tokens into fewer chunks than there are XCDs: odd numbers of chunks and
tiles, chunks of unequal length, a single chunk, repeated offsets."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,T", [(128, 128, 50, 1), (256, 256, 100, 33), (640, 1024, 400, 97), (640, 640, 250, 300),
                                     (1152, 1152, 460, 130), (2304, 768, 900, 225), (384, 4096, 1600, 65), (1024, 1024, 400, 161),
                                     (4096, 1280, 100, 64)])
def test_few_chunks(M, N, K, T):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + N + T)
    offsets[1] = offsets[-1] - max(M, N)
    off, x, dy = torch.from_numpy(offsets).cuda(), to_dev(X, "bf16"), to_dev(dY, "bf16")
    l = dd.make_layer(T, M, N, K, torch.bfloat16, dd.DD_ALGO_MATRIX)
    need = dd.dd_workspace_bytes(dd.DD_OP_BWD_WEIGHT, l)
    dV = dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_MATRIX)
    ref = orc.bwd_weight(X, dY, offsets)
    assert need >= dV.numel() * 4
    assert rel_err(to_host(dV), ref) <= TOL_DV
    assert torch.equal(dV[1], dV[K - 1])
    assert torch.equal(dV, dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_MATRIX))
