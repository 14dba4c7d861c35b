"""Products of few tokens on the matrix cores: edges of the 32- and 64-token tiles, contractions shorter than the number of
waves that share them, and groups of layers whose rows lie in several matrices."""
import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from paper_2506_11449_amd import synth
from oracle import dd_oracle as orc
from tests.parity_util import TOL, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("M,N,K,T", [
    (128, 128, 20, 1), (128, 128, 20, 33), (256, 128, 40, 65), (128, 640, 60, 31), (640, 128, 60, 64), (384, 384, 384, 32),
    (768, 768, 77, 129), (768, 768, 77, 256), (768, 768, 77, 700), (768, 768, 77, 1279), (768, 3072, 307, 63),
    (3072, 768, 307, 450), (2048, 2048, 20, 500), (4096, 1024, 205, 257), (1024, 4096, 100, 97), (4096, 4096, 30, 401)])
def test_products_of_few_tokens(M, N, K, T):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + 3 * N + T)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16")
    prepared = dd.dd_prepare(off, V, M, N)
    # the rows behind the result must stay as they are
    Y = torch.full((T + 1, N), 7.0, dtype=torch.bfloat16, device="cuda")
    dd.dd_fwd(x, None, None, N, Y=Y[:T], prepared=prepared)
    dX = torch.full((T + 1, M), 7.0, dtype=torch.bfloat16, device="cuda")
    dd.dd_bwd_input(dy, None, None, M, dX=dX[:T], prepared=prepared)
    assert (Y[T] == 7).all() and (dX[T] == 7).all()
    assert rel_err(to_host(Y[:T]), orc.fwd(X, offsets, values, N)) <= TOL["bf16"]
    assert rel_err(to_host(dX[:T]), orc.bwd_input(dY, offsets, values, M)) <= TOL["bf16"]


@pytest.mark.parametrize("M,N,K,S,T", [(128, 128, 20, 3, 5), (384, 128, 40, 2, 70), (128, 384, 40, 4, 33), (768, 768, 77, 3, 197)])
def test_groups_of_layers_with_few_tokens(M, N, K, S, T):
    cases = [random_case(M, N, K, T, "bf16", seed=11 + s) for s in range(S)]
    X = cases[0][2]
    off = torch.from_numpy(np.stack([c[0] for c in cases])).cuda()
    V = torch.stack([to_dev(c[1], "bf16") for c in cases])
    dY = torch.stack([to_dev(c[3], "bf16") for c in cases])
    prepared = dd.dd_prepare_shared(off, V, M, N)
    Y = to_host(dd.dd_fwd_shared(to_dev(X, "bf16"), prepared))
    dX = to_host(dd.dd_bwd_input_shared(dY, prepared))
    for s, (o, v, _, _) in enumerate(cases):
        assert rel_err(Y[s], orc.fwd(X, o, v, N)) <= TOL["bf16"]
    assert rel_err(dX, sum(orc.bwd_input(c[3], c[0], c[1], M) for c in cases)) <= TOL["bf16"]


@pytest.mark.parametrize("M,N,K,runs,T", [(128, 128, 1, 1, 1), (128, 384, 40, 2, 33), (384, 128, 60, 1, 200), (768, 768, 77, 1, 400),
                                          (768, 768, 300, 5, 1279), (4096, 128, 400, 3, 65), (128, 8192, 900, 8, 130),
                                          (2304, 640, 1, 1, 257)])
def test_block_skipping_with_few_tokens(M, N, K, runs, T):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=M + N + K,
                                         offsets=synth.draw_offsets_clustered(max(M, N), K, runs, seed=K))
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16")
    prepared = dd.dd_prepare(off, V, M, N)
    Y = to_host(dd.dd_fwd(x, off, None, N, prepared=prepared, algo=dd.DD_ALGO_BLOCKS))
    dX = to_host(dd.dd_bwd_input(dy, off, None, M, prepared=prepared, algo=dd.DD_ALGO_BLOCKS))
    assert rel_err(Y, orc.fwd(X, offsets, values, N)) <= TOL["bf16"]
    assert rel_err(dX, orc.bwd_input(dY, offsets, values, M)) <= TOL["bf16"]
    # blocks that no diagonal crosses are not multiplied, so what stands in their rows does not matter
    x[0, 0] = float("inf")
    crossed = np.zeros((M, N), dtype=bool)
    p = np.arange(min(M, N))
    for o in offsets:
        q = (p + o) % max(M, N)
        rows, cols = (p, q) if M <= N else (q, p)
        crossed[rows, cols] = True
    touched = np.repeat(crossed[:16].reshape(16, N // 32, 32).any(axis=(0, 2)), 32)  # 32-column blocks of contraction indices 0-15
    Y = to_host(dd.dd_fwd(x, off, None, N, prepared=prepared, algo=dd.DD_ALGO_BLOCKS))
    assert np.isfinite(Y[0][~touched]).all() and np.isfinite(Y[1:]).all()
