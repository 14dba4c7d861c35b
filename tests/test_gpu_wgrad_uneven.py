"""The matrix-core weight gradient with as many chunks of tokens as fill the chip where whole chunks per XCD would not: sizes on both
sides of the rule, the error against 64 bits, and scratch that never falls as tokens grow."""
import pytest
import torch

import paper_2506_11449_amd as dd
from tests.parity_util import TOL_DV

pytestmark = pytest.mark.gpu


# 36, 49, 40, 50 and 23 tiles; few tokens, where the chunks stay even, and more; a single slice more than chunks
@pytest.mark.parametrize("M,N,K", [(1152, 1152, 115), (896, 1792, 89), (1024, 1280, 51), (640, 2560, 60), (2944, 128, 300)])
@pytest.mark.parametrize("T", [333, 481, 3001, 13485, 20011])
def test_uneven_chunks(M, N, K, T):
    D, L = max(M, N), min(M, N)
    g = torch.Generator(device="cuda").manual_seed(M + N + T)
    X, dY = (torch.randn((T, w), device="cuda", generator=g).bfloat16() for w in (M, N))
    off = torch.randperm(D, device="cuda", generator=g)[:K].to(torch.int32)
    off[1] = off[K - 1] - D  # a repeated offset
    dV = dd.dd_bwd_weight(X, dY, off, algo=dd.DD_ALGO_MATRIX)
    p = torch.arange(L, device="cuda")[None, :]
    q = (p + off.long()[:, None]) % D
    full = X.double().t().contiguous() @ dY.double()
    ref = full[p.expand_as(q), q] if M <= N else full[q, p.expand_as(q)]
    assert ((dV.double() - ref).abs().max() / ref.abs().max()).item() <= TOL_DV
    assert torch.equal(dV[1], dV[K - 1])
    assert torch.equal(dV, dd.dd_bwd_weight(X, dY, off, algo=dd.DD_ALGO_MATRIX))


@pytest.mark.parametrize("M,N,K", [(1152, 1152, 115), (896, 1792, 89), (1024, 1280, 512), (640, 2560, 60), (2944, 128, 300), (128, 128, 100)])
def test_scratch_never_falls(M, N, K):
    need = [dd.dd_workspace_bytes(dd.DD_OP_BWD_WEIGHT, dd.make_layer(T, M, N, K, torch.bfloat16)) for T in (*range(1, 2000, 13), *range(2000, 40000, 311))]
    assert need == sorted(need)
