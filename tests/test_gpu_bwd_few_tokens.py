"""Both gradients of a layer for few tokens on the vector kernels as one launch (dd_bwd), against the CPU oracle and, bit for
bit, against the two calls."""
import pytest
import torch

import paper_2506_11449_amd as dd
from oracle import dd_oracle as orc
from tests.parity_util import TOL, TOL_DV, random_case, rel_err, to_dev, to_host

pytestmark = pytest.mark.gpu


# one token, remainders of groups and tiles, the last number of tokens it is made for and the next; diagonals shared between
# waves, more workgroups than one per diagonal, long sides either way
@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("M,N,K,T", [(1, 1, 1, 1), (64, 64, 8, 16), (65, 63, 60, 3), (63, 257, 20, 15), (300, 100, 120, 33), (257, 255, 40, 192),
                                     (257, 255, 40, 193), (1001, 77, 300, 9), (100, 1030, 31, 130), (1200, 1100, 500, 41)])
def test_both_gradients(M, N, K, T, dtype):
    offsets, values, X, dY = random_case(M, N, K, T, dtype, seed=M + N + K + T)
    off, V, x, dy = torch.from_numpy(offsets).cuda(), to_dev(values, dtype), to_dev(X, dtype), to_dev(dY, dtype)
    dX, dV = dd.dd_bwd(x, dy, off, V)
    assert rel_err(to_host(dX), orc.bwd_input(dY, offsets, values, M)) <= TOL[dtype]
    assert rel_err(to_host(dV), orc.bwd_weight(X, dY, offsets)) <= TOL_DV
    assert torch.equal(dX, dd.dd_bwd_input(dy, off, V, M)) and torch.equal(dV, dd.dd_bwd_weight(x, dy, off))


def _replays(call, repeats=20):
    call()
    torch.cuda.synchronize()
    stream, graph = torch.cuda.Stream(), torch.cuda.CUDAGraph()
    with torch.cuda.stream(stream):
        with torch.cuda.graph(graph, stream=stream):
            for _ in range(repeats):
                call()

    def us():
        a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        a.record()
        graph.replay()
        b.record()
        torch.cuda.synchronize()
        return a.elapsed_time(b) * 1e3 / repeats

    return us


# layers on which one launch took 1.2 to 1.5 times as long as two: much work, long sides, many entries
@pytest.mark.parametrize("M,N,K,T", [(519, 519, 300, 192), (6000, 1000, 20, 192), (7293, 7293, 1316, 1)])
def test_one_launch_is_not_taken_where_two_are_ahead(M, N, K, T):
    g = torch.Generator(device="cuda").manual_seed(M + N + K + T)
    r = lambda *s: torch.randn(s, device="cuda", generator=g)
    x, dy, V, off = r(T, M), r(T, N), r(K, min(M, N)), torch.randperm(max(M, N), device="cuda", generator=g)[:K].to(torch.int32)
    dX, dV, ws = torch.empty_like(x), torch.empty_like(V), dd.Workspace()
    ws.get(1 << 26, x.device)
    one = _replays(lambda: dd.dd_bwd(x, dy, off, V, dX=dX, dValues=dV, ws=ws))
    two = _replays(lambda: (dd.dd_bwd_input(dy, off, V, M, dX=dX, ws=ws), dd.dd_bwd_weight(x, dy, off, dValues=dV, ws=ws)))
    times = [(one(), two()) for _ in range(25)]  # in turn: the shortest of each
    assert min(t[0] for t in times) <= 1.15 * min(t[1] for t in times)
