"""How far the weight gradient is from the same sum in 64 bits.

Rounding an fp32 sum to nearest leaves an error of ulp / sqrt(12), 2.5e-8 of the sum's size on average over its mantissa.  An
entry is a sum of T products of random sign; its running sum grows with the square root of what has been added, so after n
additions one after the other the errors add up to 2.5e-8 * sqrt(n / 2) of the result (2-norm over the gradient)."""
import pytest
import torch

import paper_2506_11449_amd as dd

pytestmark = pytest.mark.gpu


def _error(M, N, K, T, dtype, algo):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + N + K + T)
    D, L = max(M, N), min(M, N)
    offsets = torch.sort(torch.randperm(D, device="cuda", generator=gen)[:K])[0].to(torch.int32)
    X = torch.randn((T, M), device="cuda", generator=gen).to(dtype)
    dY = torch.randn((T, N), device="cuda", generator=gen).to(dtype)
    p = torch.arange(L, device="cuda")[None, :]
    q = (p + offsets.long()[:, None]) % D
    G = X.double().t().contiguous() @ dY.double()
    ref = G[p.expand_as(q), q] if M <= N else G[q, p.expand_as(q)]
    dV = dd.dd_bwd_weight(X, dY, offsets, algo=algo).double()
    return float((dV - ref).norm() / ref.norm())


@pytest.mark.parametrize("M,N,K,T", [(768, 768, 77, 25216), (768, 768, 77, 1279), (1024, 4096, 819, 25216), (4096, 2560, 400, 788),
                                     (256, 256, 100, 6304), (128, 512, 77, 10320), (1408, 1408, 422, 1915), (2048, 2048, 200, 197)])
def test_matrix_cores(M, N, K, T):
    """No longer a chain of additions than with as many chunks as the scratch holds: two per 16 tokens of a chunk (an MFMA adds
    its sixteen products in two steps), a quarter of the chunks, four runs.  A fifth on top for the mantissas that occur."""
    l = dd.make_layer(T, M, N, K, torch.bfloat16, dd.DD_ALGO_MATRIX)
    chunks = dd.dd_workspace_bytes(dd.DD_OP_BWD_WEIGHT, l) // (4 * K * min(M, N))
    additions = T / 8 / chunks + -(-chunks // 4) + 3
    assert _error(M, N, K, T, torch.bfloat16, dd.DD_ALGO_MATRIX) <= 1.2 * 2.5e-8 * (additions / 2) ** 0.5


@pytest.mark.parametrize("M,N,K,T,dtype", [(1000, 1000, 600, 25216, torch.float32), (2000, 2000, 1000, 8192, torch.float32),
                                           (40, 3000, 3000, 9000, torch.float32), (1024, 1000, 500, 1024, torch.float32),
                                           (1536, 1528, 700, 12608, torch.bfloat16), (333, 1001, 700, 40000, torch.bfloat16),
                                           (2000, 2000, 1000, 8192, torch.bfloat16), (56, 1960, 196, 4651, torch.bfloat16)])
def test_vector_kernels(M, N, K, T, dtype):
    """At most 1024 tokens one after the other, in bf16 two tokens an addition and layers of whole 16-byte rows in at least
    eight chunks; the chunks are added in four runs, by eights.  A fifth on top for the mantissas that occur."""
    chunks = -(-T // 1024)
    if dtype == torch.bfloat16 and M % 8 == 0 and N % 8 == 0:
        chunks = max(chunks, 8)
    additions = T / chunks / (2 if dtype == torch.bfloat16 else 1) + chunks / 32 + 14
    assert _error(M, N, K, T, dtype, dd.DD_ALGO_VECTOR) <= 1.2 * 2.5e-8 * (additions / 2) ** 0.5
