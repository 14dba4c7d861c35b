"""Products on the matrix cores on the far side of the rule for few tokens, where the 64- ... 192-row tiles of 256 columns, the
128 x 128 tile and the block-skipping kernel of many tokens run, single layers and groups, with ragged token counts; and a
group in the range where it and its layers alone fall on different sides."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from paper_2506_11449_amd import synth

pytestmark = pytest.mark.gpu


def _dense(M, N, offsets, values):
    W = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    p = torch.arange(min(M, N), device="cuda")[None, :]
    q = (p + offsets.long()[:, None]) % max(M, N)
    p = p.expand_as(q)
    return W.index_put_((p, q) if M <= N else (q, p), values.double(), accumulate=True)


def _inputs(M, N, K, T, S=1, offsets=None):
    gen = torch.Generator(device="cuda")
    gen.manual_seed(M + 3 * N + 7 * T)
    D, L = max(M, N), min(M, N)
    if offsets is None:
        offsets = torch.stack([torch.randperm(D, device="cuda", generator=gen)[:K] for _ in range(S)]).to(torch.int32)
    V = (torch.randn((S, K, L), device="cuda", generator=gen) * 0.02).bfloat16()
    X = torch.randn((T, M), device="cuda", generator=gen).bfloat16()
    dY = torch.randn((S, T, N), device="cuda", generator=gen).bfloat16()
    return offsets, V, X, dY


def _close(got, ref):
    """Rounding to bf16 leaves at most 2^-8 of an element (the fp32 sum before it some 1e-6); rows are checked one by one, so
    that a wrong one does not drown in the others."""
    error, size = (got.double() - ref).norm(dim=-1), ref.norm(dim=-1)
    assert (error <= 2.0 ** -8 * size).all(), int((error > 2.0 ** -8 * size).nonzero()[0, 0])


@pytest.mark.parametrize("M,N,K,T", [(768, 768, 77, 2001), (768, 768, 77, 6305), (768, 768, 77, 9001), (768, 768, 77, 11201),
                                     (768, 768, 77, 16001), (768, 640, 60, 2001), (640, 768, 60, 5001), (640, 384, 60, 3001),
                                     (128, 128, 20, 4001), (896, 128, 90, 6001), (1024, 4096, 200, 801)])
def test_single_layers_beyond_few_tokens(M, N, K, T):
    offsets, V, X, dY = _inputs(M, N, K, T)
    W = _dense(M, N, offsets[0], V[0])
    prepared = dd.dd_prepare(offsets[0], V[0], M, N)
    Y = torch.full((T + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
    dX = torch.full((T + 1, M), 7.0, dtype=torch.bfloat16, device="cuda")
    dd.dd_fwd(X, None, None, N, Y=Y[:T], prepared=prepared)
    dd.dd_bwd_input(dY[0], None, None, M, dX=dX[:T], prepared=prepared)
    assert (Y[T] == 7).all() and (dX[T] == 7).all()
    _close(Y[:T], X.double() @ W)
    _close(dX[:T], dY[0].double() @ W.t().contiguous())


@pytest.mark.parametrize("M,N,K,S,T", [(128, 384, 40, 2, 1001), (128, 384, 40, 2, 2001), (128, 384, 40, 2, 8001), (128, 384, 40, 2, 12001),
                                       (768, 640, 60, 2, 1001), (768, 640, 60, 2, 2001), (768, 640, 60, 2, 8001),
                                       (768, 640, 60, 2, 12001), (384, 384, 40, 3, 1001), (384, 384, 40, 3, 6001)])
def test_groups_beyond_few_tokens(M, N, K, S, T):
    """Tiles of 256 columns that a matrix boundary cuts where 256 does not divide the width."""
    offsets, V, X, dY = _inputs(M, N, K, T, S)
    prepared = dd.dd_prepare_shared(offsets, V, M, N)
    Y, dX = dd.dd_fwd_shared(X, prepared), dd.dd_bwd_input_shared(dY, prepared)
    Ws = [_dense(M, N, offsets[s], V[s]) for s in range(S)]
    for s in range(S):
        _close(Y[s], X.double() @ Ws[s])
    _close(dX, sum(dY[s].double() @ Ws[s].t().contiguous() for s in range(S)))


@pytest.mark.parametrize("M,N,S,T", [(768, 768, 3, 800), (1024, 1024, 3, 700), (128, 384, 2, 800)])
def test_a_group_and_its_layers_alone_in_different_kernels(M, N, S, T):
    """The sums are made in another order, so the results agree within their rounding and need not be the same bits."""
    offsets, V, X, dY = _inputs(M, N, max(M, N) // 10, T, S)
    Y = dd.dd_fwd_shared(X, dd.dd_prepare_shared(offsets, V, M, N))
    for s in range(S):
        alone = dd.dd_fwd(X, None, None, N, prepared=dd.dd_prepare(offsets[s], V[s], M, N))
        ref = X.double() @ _dense(M, N, offsets[s], V[s])
        _close(Y[s], ref)
        _close(alone, ref)
        differ = (Y[s] != alone).float().mean()  # only where the fp32 sums straddle a rounding boundary
        assert differ < 1e-2


@pytest.mark.parametrize("kind", ["runs", "wrapped", "uniform", "dense"])
@pytest.mark.parametrize("M,N,T", [(768, 768, 2688), (768, 768, 2689), (768, 768, 2801), (3072, 768, 2801), (768, 3072, 2801), (384, 1152, 5501),
                                   (1152, 384, 5501), (8192, 256, 8201), (256, 8192, 2001)])
def test_block_skipping_beyond_few_tokens(M, N, T, kind):
    """768^2 has 504 and 516 tiles of 64 x 64 at 2688 and 2689 tokens, either side of the rule."""
    D = max(M, N)
    K = {"runs": D // 10, "wrapped": D // 12, "uniform": D // 16, "dense": D}[kind]
    offsets = {"runs": lambda: synth.draw_offsets_clustered(D, K, 3, seed=T), "wrapped": lambda: np.arange(K) - K // 2,
               "uniform": lambda: np.random.default_rng(T).permutation(D)[:K], "dense": lambda: np.arange(D)}[kind]()
    offsets = torch.from_numpy(np.asarray(offsets, dtype=np.int32)).cuda()[None]
    offsets, V, X, dY = _inputs(M, N, K, T, offsets=offsets)
    W = _dense(M, N, offsets[0], V[0])
    prepared = dd.dd_prepare(offsets[0], V[0], M, N)
    Y = torch.full((T + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
    dX = torch.full((T + 1, M), 7.0, dtype=torch.bfloat16, device="cuda")
    dd.dd_fwd(X, offsets[0], None, N, Y=Y[:T], prepared=prepared, algo=dd.DD_ALGO_BLOCKS)
    dd.dd_bwd_input(dY[0], offsets[0], None, M, dX=dX[:T], prepared=prepared, algo=dd.DD_ALGO_BLOCKS)
    assert (Y[T] == 7).all() and (dX[T] == 7).all()
    _close(Y[:T], X.double() @ W)
    _close(dX[:T], dY[0].double() @ W.t().contiguous())
