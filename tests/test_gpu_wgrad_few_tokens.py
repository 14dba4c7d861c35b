"""The weight gradient straight from memory: remainders of its blocks of sixteen and four tokens, either side of the rule that
takes it (T <= 192 and T * K * L <= 3e7), wide layers that never use a tile, inputs that are not finite."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", [(65, 63, 9, 1), (65, 63, 9, 3), (64, 64, 8, 4), (63, 257, 20, 15), (257, 256, 20, 16), (257, 300, 31, 17),
                                     (100, 100, 100, 33), (70, 90, 12, 192), (70, 90, 12, 193), (1000, 900, 181, 184), (1000, 900, 181, 185),
                                     (24, 10300, 12, 2051), (10300, 24, 12, 3000), (9000, 8999, 5, 1030)])
def test_few_tokens_and_wide_layers(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + 7 * N + T)
    offsets[0] -= max(M, N)
    off, x, dy = torch.from_numpy(offsets).cuda(), to_dev(X, dtype), to_dev(dY, dtype)
    dV = dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_VECTOR)
    assert rel_err(to_host(dV), orc.bwd_weight(X, dY, offsets)) <= TOL_DV
    x[T - 1, 0], dy[0, N - 1] = float("inf"), float("nan")  # reach the entries that multiply them and no others
    got = dd.dd_bwd_weight(x, dy, off, algo=dd.DD_ALGO_VECTOR)
    p, q = np.arange(min(M, N))[None, :], (np.arange(min(M, N))[None, :] + offsets[:, None]) % max(M, N)
    rows, cols = (p + 0 * q, q) if M <= N else (q, p + 0 * q)
    touched = torch.from_numpy((rows == 0) | (cols == N - 1)).cuda()
    assert torch.equal(got[~touched], dV[~touched]) and not torch.isfinite(got[touched]).any()


def test_more_than_a_thousand_million_values():
    """K * L beyond 2^30: every entry of the sum over the chunks has a workgroup (4.4 GB of gradient, 8.7 GB of scratch)."""
    D, T = 33000, 1025
    gen = torch.Generator(device="cuda")
    gen.manual_seed(1)
    offsets = torch.randperm(D, device="cuda", generator=gen).to(torch.int32)
    X, dY = (torch.randn((T, D), device="cuda", generator=gen) for _ in range(2))
    dV = torch.full((D, D), float("nan"), device="cuda")
    dd.dd_bwd_weight(X, dY, offsets, dValues=dV, ws=dd.Workspace())
    k, p = (torch.randint(0, D, (4000,), device="cuda", generator=gen) for _ in range(2))
    k[:2], p[:2] = torch.tensor([0, D - 1]), torch.tensor([0, D - 1])
    q = (p + offsets[k].long()) % D
    ref = (X[:, p].double() * dY[:, q].double()).sum(0)
    assert float((dV[k, p].double() - ref).norm() / ref.norm()) <= 1e-6
    assert not torch.isnan(dV.sum(1)).any()
