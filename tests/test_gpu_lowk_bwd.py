"""Both gradients of a layer with a handful of diagonals as one kernel (dd_bwd), against the CPU oracle and, bit for bit,
against the two calls."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


# one token, less than a tile, remainders of tiles; every number of diagonals it is made for, and the first it is not; one, two
# and four column pairs a lane; layers that contract (two kernels)
@pytest.mark.parametrize("M,N,K,T", [(128, 128, 1, 1), (128, 256, 8, 5), (256, 384, 7, 37), (384, 384, 2, 300), (1024, 2048, 8, 1003),
                                     (1024, 1024, 4, 4097), (640, 1024, 5, 513), (2048, 2048, 3, 70), (4096, 4096, 6, 131),
                                     (3072, 3072, 2, 1001), (768, 3072, 9, 200), (1024, 512, 3, 333)])
@pytest.mark.parametrize("algo", ["vector", "auto"])
def test_both_gradients(M, N, K, T, algo):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + N + K + T)
    offsets = offsets - max(M, N) * (np.arange(K) % 3 - 1).astype(offsets.dtype)  # any representative counts
    if K > 4:
        offsets[K - 1] = offsets[0]  # repeated
    off, x, dy = torch.from_numpy(offsets).cuda(), to_dev(X, "bf16"), to_dev(dY, "bf16")
    flat = torch.empty(values.size + 1, dtype=torch.bfloat16, device="cuda")
    V = flat[1:].view(values.shape)  # values may start at any element
    V.copy_(to_dev(values, "bf16"))
    a = dd.DD_ALGO_VECTOR if algo == "vector" else dd.DD_ALGO_AUTO
    dX, dV = dd.dd_bwd(x, dy, off, V, algo=a)
    assert rel_err(to_host(dX), orc.bwd_input(dY, offsets, values, M)) <= TOL["bf16"]
    assert rel_err(to_host(dV), orc.bwd_weight(X, dY, offsets)) <= TOL_DV
    assert torch.equal(dX.view(torch.int16), dd.dd_bwd_input(dy, off, V, M, algo=a).view(torch.int16))
    assert torch.equal(dV, dd.dd_bwd_weight(x, dy, off, algo=a))
    again = dd.dd_bwd(x, dy, off, V, algo=a)
    assert torch.equal(dX.view(torch.int16), again[0].view(torch.int16)) and torch.equal(dV, again[1])


# layers where one of the two calls, both or neither run on the matrix cores under DD_ALGO_AUTO
@pytest.mark.parametrize("M,N,K,T", [(512, 512, 8, 3000), (1024, 1024, 8, 2000), (256, 256, 6, 4000), (768, 768, 6, 9000), (1024, 2048, 7, 2000),
                                     (1024, 1024, 4, 2000), (2048, 2048, 8, 900)])
def test_scratch_does_not_choose_the_kernel(M, N, K, T):
    """The scratch that the library asks for, ten times as much, and the two calls: one result, bit for bit."""
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + N + K + T)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16")
    need = dd.dd_workspace_bytes(dd.DD_OP_BWD, dd.make_layer(T, M, N, K, torch.bfloat16, dd.DD_ALGO_AUTO))
    results = []
    for size in (need, 10 * need):
        ws = dd.Workspace()
        ws.get(size, x.device)
        results.append(dd.dd_bwd(x, dy, off, V, ws=ws))
    results.append((dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_weight(x, dy, off)))
    for dX, dV in results[1:]:
        assert torch.equal(dX.view(torch.int16), results[0][0].view(torch.int16)) and torch.equal(dV, results[0][1])
