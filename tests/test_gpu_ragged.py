"""Layers whose widths are multiples of eight but not of 128 on the matrix cores (bf16, DD_ALGO_AUTO, from some hundred tokens on),
against 64 bits, or against the vector kernels (which are compared with the oracle) where it is about numbers that are not finite.
Every shape says which of its three products run there -- f(orward), b(ackward-input), g(radient) -- by the library's own rules."""
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


def _families(M, N, K, T):
    """Which products the library's rules send to the matrix cores."""
    lib, D, L = binding.load_library(), max(M, N), min(M, N)

    def says(name, *sizes, masked=None):
        rule = lib[name]
        rule.restype, rule.argtypes = ctypes.c_bool, [ctypes.c_int64] + 3 * [ctypes.c_int] + [ctypes.c_bool] * (masked is not None)
        return rule(*sizes, *([] if masked is None else [masked]))

    product = lambda masked: all(says(f"_ZN2dd{name}Eliiib", T, D, L, K, masked=masked)
                                 for name in ("19product_ragged_pays", "24product_ragged_ever_pays"))
    gradient = says("_ZN2dd23weight_grad_ragged_paysEliii", T, D, L, K)
    return "".join(name for name, there in (("f", product(M <= N)), ("b", product(M > N)), ("g", gradient)) if there)


def _case(M, N, K, T, seed=0):
    offsets, values, X, dY = random_case(M, N, K, T, "bf16", seed=seed + M + N + K + T)
    return (offsets, values, X, dY), (torch.from_numpy(offsets).cuda(), to_dev(values, "bf16"), to_dev(X, "bf16"), to_dev(dY, "bf16"))


def _exact(x, dy, off, V, M, N):
    """The three products in 64 bits."""
    D, L = max(M, N), min(M, N)
    p = torch.arange(L, device="cuda")[None, :].expand(V.shape)
    q = (p + off.long()[:, None]) % D
    at = (p, q) if M <= N else (q, p)
    W = torch.zeros((M, N), dtype=torch.float64, device="cuda")
    W.index_put_(at, V.double(), accumulate=True)
    return x.double() @ W, dy.double() @ W.t().contiguous(), (x.double().t().contiguous() @ dy.double())[at]


# every tile of the products; remainders of eight columns and of one token; more candidates than tiles along either side; narrow sides
@pytest.mark.parametrize("M,N,K,T,runs", [(392, 376, 392, 601, "b"), (264, 520, 208, 1000, "f"), (1048, 136, 1048, 1500, "fb"), (264, 264, 105, 5005, "fb"),
                                          (1048, 136, 419, 2049, "fb"), (776, 768, 310, 1001, "fb"), (520, 520, 208, 12608, "fbg"),
                                          (1496, 1496, 149, 5005, "fbg"), (1496, 1400, 598, 12607, "fbg"), (8, 264, 13, 5005, "g"),
                                          (264, 24, 264, 5001, ""), (768, 776, 776, 257, "fb"), (520, 104, 423, 6340, "fbg"), (1000, 320, 400, 2000, "fbg")])
def test_products_and_gradient(M, N, K, T, runs):
    assert _families(M, N, K, T) == runs
    (offsets, values, X, dY), (off, V, x, dy) = _case(M, N, K, T)
    offsets -= max(M, N) * (np.arange(K) % 3 - 1).astype(offsets.dtype)  # any representative counts
    off = torch.from_numpy(offsets).cuda()
    Y, (dX, dV) = dd.dd_fwd(x, off, V, N), dd.dd_bwd(x, dy, off, V)
    if M * N * T < 400000000:
        refs = orc.fwd(X, offsets, values, N), orc.bwd_input(dY, offsets, values, M), orc.bwd_weight(X, dY, offsets)
    else:
        refs = [a.cpu().numpy() for a in _exact(x, dy, off, V, M, N)]
    for got, ref, tol in zip((Y, dX, dV), refs, (TOL["bf16"], TOL["bf16"], TOL_DV)):
        assert rel_err(to_host(got), ref) <= tol
    assert torch.equal(dX, dd.dd_bwd_input(dy, off, V, M)) and torch.equal(dV, dd.dd_bwd_weight(x, dy, off))


# the window of offsets that cross a tile (383 of them) wider than the candidates: from the smallest side on, tiles of 192 x 192 and
# of 128 x 256, expanding and contracting, an offset given twice
@pytest.mark.parametrize("M,N,K,T", [(8, 256, 4, 3027), (256, 232, 12, 8000), (232, 256, 12, 8000), (264, 168, 132, 12608), (136, 264, 4, 2172),
                                     (328, 328, 328, 6001), (376, 376, 94, 3000), (360, 376, 94, 5005)])
def test_gradient_of_tiles_that_wrap(M, N, K, T):
    assert "g" in _families(M, N, K, T)
    _, (off, V, x, dy) = _case(M, N, K, T)
    if K < max(M, N):
        off[K - 1] = off[0]
    ref = _exact(x, dy, off, V, M, N)[2].cpu().numpy()
    got, vector = dd.dd_bwd_weight(x, dy, off), dd.dd_bwd_weight(x, dy, off, algo=VECTOR)
    assert not torch.equal(got, vector)  # sums in another order: another family ran
    got = got.cpu().numpy()
    assert rel_err(got, ref) <= TOL_DV
    # entry by entry as well: a misplaced one is of the size of all others.  (T products of two normals: their sum is sqrt(T) large and
    # its error below T / 16 additions in fp32 of sums of up to 4 sqrt(T))
    assert np.abs(got - ref).max() <= 4 * np.sqrt(T) * (T / 16) * 2.0 ** -24


@pytest.mark.parametrize("M,N,K,T,runs", [(392, 376, 392, 601, "b"), (264, 264, 105, 5005, "fb"), (1000, 320, 400, 2000, "fbg"), (1048, 136, 419, 2049, "fb"),
                                          (776, 768, 310, 1001, "fb"), (520, 104, 423, 6340, "fbg"), (520, 520, 208, 12608, "fbg"),
                                          (1496, 1496, 149, 5005, "fbg"), (1496, 1400, 598, 12607, "fbg"), (256, 232, 12, 8000, "g")])
def test_inputs_that_are_not_finite_reach_their_own_diagonals_only(M, N, K, T, runs):
    assert _families(M, N, K, T) == runs
    _, (off, V, x, dy) = _case(M, N, K, T)
    for a in (x, dy):
        a[0, 3], a[T - 1, -1], a[T // 2, 0] = float("inf"), float("nan"), float("-inf")
        a[T // 4:T // 4 + 19, 7] = float("inf")  # more tokens of a tile than are taken at a time
    V[K // 2, 5] = float("inf")
    for got, ref in ((dd.dd_fwd(x, off, V, N), dd.dd_fwd(x, off, V, N, algo=VECTOR)),
                     (dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR)),
                     (dd.dd_bwd_weight(x, dy, off), dd.dd_bwd_weight(x, dy, off, algo=VECTOR))):
        got, ref = to_host(got), to_host(ref)
        finite = np.isfinite(ref)
        assert (np.isfinite(got) == finite).all() and finite.any() and not finite.all()
        assert (np.isnan(got) == np.isnan(ref)).all() and (np.sign(got[np.isinf(ref)]) == np.sign(ref[np.isinf(ref)])).all()
        assert rel_err(got[finite], ref[finite]) <= TOL["bf16"]


@pytest.mark.parametrize("M,N,K,T", [(264, 264, 105, 5005), (1000, 320, 400, 2000)])
def test_nothing_finite(M, N, K, T):
    _, (off, V, x, dy) = _case(M, N, K, T)
    x.fill_(float("nan"))
    dy.fill_(float("inf"))
    assert dd.dd_fwd(x, off, V, N).isnan().sum() == dd.dd_fwd(x, off, V, N, algo=VECTOR).isnan().sum()
    got, ref = dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR)
    assert torch.equal(got.isnan(), ref.isnan()) and torch.equal(got[~got.isnan()], ref[~ref.isnan()])


def _us(call):
    call()
    times = []
    for _ in range(15):
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        call()
        b.record()
        torch.cuda.synchronize()
        times.append(a.elapsed_time(b) * 1e3)
    return min(times)


def test_a_number_that_is_not_finite_costs_its_token_only():
    """One token in a thousand with such a number: the product stays well ahead of the vector kernels (115-125 and 650 us)."""
    M, N, K, T = 1496, 1496, 598, 12608
    _, (off, V, x, dy) = _case(M, N, K, T)
    x[::1000, 3] = float("nan")
    Y, ws = torch.empty_like(dy), dd.Workspace()
    assert _us(lambda: dd.dd_fwd(x, off, V, N, Y=Y, ws=ws)) <= 0.5 * _us(lambda: dd.dd_fwd(x, off, V, N, Y=Y, ws=ws, algo=VECTOR))


@pytest.mark.parametrize("M,N,K,T", [(392, 376, 392, 601), (264, 264, 105, 5005), (1000, 320, 400, 2000)])
def test_repeated_offsets_cost_no_precision(M, N, K, T):
    """Half of the offsets given three times: against 64 bits the products are as exact as those of the vector kernels, which add the
    products of every copy (a single rounding of the summed weights to bf16 would make the error half as large again)."""
    _, (off, V, x, dy) = _case(M, N, K, T)
    off[K // 4:K // 2] = off[:K // 2 - K // 4]
    off[K // 2:K // 2 + K // 4] = off[:K // 4]
    exact = _exact(x, dy, off, V, M, N)
    for got, vector, ref in ((dd.dd_fwd(x, off, V, N), dd.dd_fwd(x, off, V, N, algo=VECTOR), exact[0]),
                             (dd.dd_bwd_input(dy, off, V, M), dd.dd_bwd_input(dy, off, V, M, algo=VECTOR), exact[1])):
        assert (got.double() - ref).norm() <= 1.01 * (vector.double() - ref).norm()


@pytest.mark.parametrize("M,N,K,T,runs", [(392, 376, 392, 601, "b"), (264, 264, 105, 5005, "fb"), (1000, 320, 400, 2000, "fbg"), (1496, 1496, 1496, 3000, "fbg")])
def test_copies_of_an_offset_add_in_order(M, N, K, T, runs):
    """Weights of 1e30, -1e30 and about one on one offset: added in the order of the diagonals their sum is the last, exactly; in another
    order nothing is left of it.  (1496 diagonals are looked at in two passes.)"""
    assert _families(M, N, K, T) == runs
    _, (off, V, x, dy) = _case(M, N, K, T)
    n = K // 6  # triples from positions far apart
    off[n:2 * n] = off[:n]
    off[K - n:] = off[:n]
    V[:n], V[n:2 * n] = 1e30, -1e30
    small = V.clone()
    small[:2 * n] = 0
    exact = _exact(x, dy, off, small, M, N)
    Y, dX = dd.dd_fwd(x, off, V, N), dd.dd_bwd_input(dy, off, V, M)
    if "f" in runs:
        assert rel_err(to_host(Y), exact[0].cpu().numpy()) <= TOL["bf16"]
    if "b" in runs:
        assert rel_err(to_host(dX), exact[1].cpu().numpy()) <= TOL["bf16"]
    for _ in range(3):
        assert torch.equal(Y, dd.dd_fwd(x, off, V, N)) and torch.equal(dX, dd.dd_bwd_input(dy, off, V, M))


@pytest.mark.parametrize("M,N,K,T,runs", [(264, 264, 105, 5005, "fb"), (1000, 320, 400, 2000, "fbg"), (392, 376, 392, 601, "b")])
def test_copies_whose_sum_leaves_the_range(M, N, K, T, runs):
    """Two weights of 2e38 on one offset, inputs so small that their products are finite: so are the results."""
    assert _families(M, N, K, T) == runs
    _, (off, V, x, dy) = _case(M, N, K, T)
    off[K - 1] = off[0]
    V[0] = V[K - 1] = 2e38
    x, dy = (x * 1e-3).bfloat16(), (dy * 1e-3).bfloat16()
    exact = _exact(x, dy, off, V, M, N)
    for got, ref in ((dd.dd_fwd(x, off, V, N), exact[0]), (dd.dd_bwd_input(dy, off, V, M), exact[1])):
        assert torch.isfinite(got).all() and rel_err(to_host(got), ref.cpu().numpy()) <= TOL["bf16"]


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
