"""Calls without a workspace on several streams and threads and in graphs: each has scratch of its own.  The layers are such that the
products build their operand in scratch (bf16, widths that are multiples of eight)."""
import threading

import pytest
import torch

import paper_2506_11449_amd as dd

pytestmark = pytest.mark.gpu

M, N, K, T = 520, 392, 60, 4000


def _layer(seed):
    g = torch.Generator(device="cuda")
    g.manual_seed(seed)
    r = lambda *s: torch.randn(s, device="cuda", generator=g).bfloat16()
    off = torch.sort(torch.randperm(M, device="cuda", generator=g)[:K])[0].to(torch.int32)
    return r(T, M), r(T, N), off, r(K, N)


def _step(X, dY, off, V, stream=None):
    return (dd.dd_fwd(X, off, V, N, stream=stream), *dd.dd_bwd(X, dY, off, V, stream=stream))


def _same(got, ref):
    return all(torch.equal(a, b) for a, b in zip(got, ref))


def test_streams():
    layers = [_layer(i) for i in range(4)]
    refs = [_step(*l) for l in layers]
    streams = [torch.cuda.Stream() for _ in layers]
    torch.cuda.synchronize()
    got = []
    for _ in range(20):
        for l, s in zip(layers, streams):
            with torch.cuda.stream(s):
                got.append(_step(*l))
    torch.cuda.synchronize()
    assert all(_same(g, refs[i % 4]) for i, g in enumerate(got))


def test_a_stream_that_is_named():
    """Outputs of the caller's own: what is allocated here belongs to the current stream."""
    layers, streams = [_layer(i) for i in range(2)], [torch.cuda.Stream() for _ in range(2)]
    refs = [dd.dd_fwd(X, off, V, N) for X, _, off, V in layers]
    out = [[torch.empty_like(r) for _ in range(20)] for r in refs]
    torch.cuda.synchronize()
    for i in range(20):
        for (X, _, off, V), s, Y in zip(layers, streams, out):
            dd.dd_fwd(X, off, V, N, Y=Y[i], stream=s)
    torch.cuda.synchronize()
    assert all(torch.equal(Y, r) for Ys, r in zip(out, refs) for Y in Ys)


def test_threads_on_one_stream():
    layers = [_layer(i) for i in range(4)]
    refs, got = [_step(*l) for l in layers], [[] for _ in layers]
    torch.cuda.synchronize()

    def work(i):
        for _ in range(20):
            got[i].append(_step(*layers[i]))

    workers = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for w in workers:
        w.start()
    for w in workers:
        w.join()
    torch.cuda.synchronize()
    assert all(_same(g, ref) for results, ref in zip(got, refs) for g in results)


def test_a_captured_call_keeps_its_block():
    layer, other = _layer(1), _layer(2)
    ref = _step(*layer)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        captured = _step(*layer)
    for _ in range(3):
        for t in captured:
            t.zero_()
        graph.replay()
        eager = _step(*other)  # while the graph runs on
        wide = torch.randn(2000, 1000, device="cuda").bfloat16()  # and a call that needs a larger block
        dd.dd_fwd(wide, torch.arange(300, dtype=torch.int32, device="cuda"), torch.ones(300, 1000, dtype=torch.bfloat16, device="cuda"), 1000)
        torch.cuda.synchronize()
        assert _same(captured, ref) and _same(eager, _step(*other))
