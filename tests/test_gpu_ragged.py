"""Layers whose widths are multiples of eight but not of 128 on the matrix cores (bf16, DD_ALGO_AUTO, from some hundred tokens on),
against the CPU oracle, or against the vector kernels (which are) where that would take too long."""
import ctypes

import numpy as np
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from paper_2506_11449_amd import binding
from tests.parity_util import TOL, TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu

VECTOR = dd.DD_ALGO_VECTOR


def _case(M, N, K, T, seed=0):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=seed + M + N + K + T)
    return (offsets, values, X, dY), (torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16"))


# every tile of the products; remainders of eight columns and of one token; more candidates than tiles along either side; narrow sides
@pytest.mark.parametrize("M,N,K,T", [(392, 376, 392, 601), (264, 520, 208, 1000), (1048, 136, 1048, 1500), (264, 264, 105, 5005),
                                     (1048, 136, 419, 2049), (776, 768, 310, 1001), (520, 520, 208, 12608), (1496, 1496, 149, 5005),
                                     (1496, 1400, 598, 12607), (8, 264, 13, 5005), (264, 24, 264, 5001), (768, 776, 776, 257)])
def test_products_and_gradient(M, N, K, T):
    (offsets, values, X, dY), (off, V, x, dy) = _case(M, N, K, T)
    offsets -= max(M, N) * (np.arange(K) % 3 - 1).astype(offsets.dtype)  # any representative counts
    off = torch.from_numpy(offsets).cuda()
    Y, (dX, dV) = dd.dd_fwd(x, off, V, N), dd.dd_bwd(x, dy, off, V)
    if M * N * T < 400000000:
        refs = orc.fwd(X, offsets, values, N), orc.bwd_input(dY, offsets, values, M), orc.bwd_weight(X, dY, offsets)
    else:
        refs = [to_host(a) for a in (dd.dd_fwd(x, off, V, N, algo=VECTOR), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR),
                                     dd.dd_bwd_weight(x, dy, off, algo=VECTOR))]
    for got, ref, tol in zip((Y, dX, dV), refs, (TOL["bf16"], TOL["bf16"], TOL_DV)):
        assert rel_err(to_host(got), ref) <= tol
    assert torch.equal(dX, dd.dd_bwd_input(dy, off, V, M)) and torch.equal(dV, dd.dd_bwd_weight(x, dy, off))


@pytest.mark.parametrize("M,N,K,T", [(392, 376, 392, 601), (264, 264, 105, 5005), (1000, 320, 400, 2000)])
def test_inputs_that_are_not_finite_reach_their_own_diagonals_only(M, N, K, T):
    _, (off, V, x, dy) = _case(M, N, K, T)
    for a in (x, dy):
        a[0, 3], a[T - 1, -1], a[T // 2, 0] = float("inf"), float("nan"), float("-inf")
    V[K // 2, 5] = float("inf")
    for got, ref in ((dd.dd_fwd(x, off, V, N), dd.dd_fwd(x, off, V, N, algo=VECTOR)),
                     (dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR)),
                     (dd.dd_bwd_weight(x, dy, off), dd.dd_bwd_weight(x, dy, off, algo=VECTOR))):
        got, ref = to_host(got), to_host(ref)
        finite = np.isfinite(ref)
        assert (np.isfinite(got) == finite).all() and finite.any() and not finite.all()
        assert rel_err(got[finite], ref[finite]) <= TOL["bf16"]


@pytest.mark.parametrize("M,N,K,T", [(392, 376, 392, 601), (264, 264, 105, 5005), (1000, 320, 400, 2000)])
def test_repeated_offsets_cost_no_precision(M, N, K, T):
    """Half of the offsets given three times: against 64 bits the products are as exact as those of the vector kernels, which add the
    products of every copy (a single rounding of the summed weights to bf16 would make the error half as large again)."""
    _, (off, V, x, dy) = _case(M, N, K, T)
    off[K // 4:K // 2] = off[:K // 2 - K // 4]
    off[K // 2:K // 2 + K // 4] = off[:K // 4]
    D, L = max(M, N), min(M, N)
    p = torch.arange(L, device="cuda")
    q = (p[None, :] + off.long()[:, None]) % D
    pp = p[None, :].expand_as(q)
    W = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    W.index_put_((pp, q) if M <= N else (q, pp), V.double(), accumulate=True)
    for got, vector, ref in ((dd.dd_fwd(x, off, V, N), dd.dd_fwd(x, off, V, N, algo=VECTOR), x.double() @ W),
                             (dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR), dy.double() @ W.t().contiguous())):
        assert (got.double() - ref).norm() <= 1.01 * (vector.double() - ref).norm()


def test_without_scratch_the_vector_kernels_serve():
    M, N, K, T = 264, 264, 105, 5005
    _, (off, V, x, dy) = _case(M, N, K, T)
    layer = dd.make_layer(T, M, N, K, torch.bfloat16, dd.DD_ALGO_AUTO)
    assert dd.dd_workspace_bytes(dd.DD_OP_FWD, layer) > 0
    lib, Y = binding.load_library(), torch.empty((T, N), dtype=torch.bfloat16, device="cuda")
    stream = torch.cuda.current_stream().cuda_stream
    assert lib.dd_fwd(ctypes.byref(layer), x.data_ptr(), off.data_ptr(), V.data_ptr(), Y.data_ptr(), None, 0, stream) == 0
    assert torch.equal(Y, dd.dd_fwd(x, off, V, N, algo=VECTOR))
    odd = torch.empty(T * M + 1, dtype=torch.bfloat16, device="cuda")[1:].view(T, M)  # not 16-byte aligned
    odd.copy_(x)
    assert torch.equal(dd.dd_fwd(odd, off, V, N), Y)
