"""The ends of bf16's range: subnormal inputs, weights and results count in every kernel family, and the rounding of what leaves
(by the hardware's conversion) is to nearest even with NaN kept, whatever its payload."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd

pytestmark = pytest.mark.gpu

SMALLEST = 2.0 ** -133  # the step between bf16 subnormals


def _case(M, N, K, T, x, v, g):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K + T)
    D, L = max(M, N), min(M, N)
    normal = lambda scale, *shape: (torch.randn(shape, device="cuda", generator=gen, dtype=torch.float64) * scale).bfloat16()
    offsets = torch.sort(torch.randperm(D, device="cuda", generator=gen)[:K])[0].to(torch.int32)
    V, X, dY = normal(v, K, L), normal(x, T, M), normal(g, T, N)
    p = torch.arange(L, device="cuda")[None, :]
    q = (p + offsets.long()[:, None]) % D
    at = (p.expand_as(q), q) if M <= N else (q, p.expand_as(q))
    W = torch.zeros((M, N), dtype=torch.float64, device="cuda").index_put_(at, V.double(), accumulate=True)
    return offsets, V, X, dY, X.double() @ W, dY.double() @ W.t().contiguous(), (X.double().t().contiguous() @ dY.double())[at]


# subnormal inputs; subnormal weights and gradients; subnormal results
@pytest.mark.parametrize("x,v,g", [(1e-39, 1e30, 1e5), (1e20, 1e-39, 1e-39), (1e-20, 1e-19, 1e-20)])
@pytest.mark.parametrize("M,N,K,T,algo", [(100, 260, 31, 50, "vector"), (257, 255, 40, 300, "vector"), (104, 264, 32, 50, "vector"),
                                          (256, 384, 40, 50, "matrix"), (256, 384, 40, 3000, "matrix"), (256, 384, 4, 300, "vector")])
def test_subnormal_numbers_count(M, N, K, T, algo, x, v, g):
    algo = {"vector": dd.DD_ALGO_VECTOR, "matrix": dd.DD_ALGO_MATRIX}[algo]
    offsets, V, X, dY, Y_ref, dX_ref, dV_ref = _case(M, N, K, T, x, v, g)
    Y, dX = dd.dd_fwd(X, offsets, V, N, algo=algo), dd.dd_bwd_input(dY, offsets, V, M, algo=algo)
    for got, ref in ((Y, Y_ref), (dX, dX_ref)):
        # half a unit of the result: 2^-9 ... 2^-8 of it, or half a subnormal step; then the fp32 sum, 2^-24 an addition of
        # up to K terms of the result's size and half an fp32 subnormal step each
        bound = 2.0 ** -8 * ref.abs() + 0.5 * SMALLEST + K * (2.0 ** -24 * ref.abs().max() + 2.0 ** -150)
        assert ((got.double() - ref).abs() <= bound).all()
    dV = dd.dd_bwd_weight(X, dY, offsets, algo=algo).double()
    assert ((dV - dV_ref).abs() <= T * (2.0 ** -24 * dV_ref.abs().max() + 2.0 ** -150)).all()


def test_rounding_to_bf16():
    bits = np.array([0x7f800001, 0x7f80ffff, 0x7fc00000, 0xffc00001, 0xff800001, 0x7f800000, 0xff800000, 0x00000001, 0x00007fff, 0x00008000,
                     0x00008001, 0x00018000, 0x80008001, 0x007fffff, 0x3f808000, 0x3f808001, 0x3f818000, 0x7f7f7fff, 0x7f7f8000,
                     0xff7fffff, 0x80000000], dtype=np.uint32)
    alpha = torch.from_numpy(bits.view(np.float32)).cuda()
    n, L = len(bits), 8
    V = torch.ones((n, L), dtype=torch.bfloat16, device="cuda")  # alpha * 1 is alpha: what is left is the rounding
    out = dd.dd_scale_values(torch.arange(n, dtype=torch.int32, device="cuda"), alpha, V).view(torch.int16)
    got = out.cpu().numpy().view(np.uint16)
    nan = (bits & 0x7fffffff) > 0x7f800000
    expected = ((bits.astype(np.uint64) + 0x7fff + ((bits >> 16) & 1)) >> 16).astype(np.uint16)
    assert (got[~nan] == expected[~nan][:, None]).all()
    assert ((got[nan] & 0x7fff) > 0x7f80).all() and ((got[nan] & 0x40) != 0).all()  # NaN, quiet
