"""The binding's short way (csrc/fastcall.cpp) against its long way: the same results bit for bit, and to anything but a plain call
(exact contiguous GPU tensors of the right type and shape, the workspace large enough) the answer None, which leaves the
call to the checks in Python."""
import pytest
import torch

import paper_2506_11449_amd as dd
from paper_2506_11449_amd import binding

pytestmark = pytest.mark.gpu


class _Declines:
    def __getattr__(self, name):
        return lambda *a: None


def _layer(T, M, N, K, dtype):
    g = torch.Generator().manual_seed(T + M + N + K)
    D, L = max(M, N), min(M, N)
    r = lambda *s: torch.randn(s, generator=g).to(dtype).cuda()
    scores = torch.randn((1, D), generator=g).cuda()
    return r(T, M), r(T, N), r(K, L), scores


def _calls(X, dY, V, scores, ws, stream=None, given=True):
    """Every entry point with a short way, outputs given or not: the list of what they return."""
    (T, M), N, K, L, D = X.shape, dY.shape[1], V.shape[0], V.shape[1], scores.shape[1]
    new = lambda shape, like: torch.full(shape, 7, dtype=like, device="cuda") if given else None
    i32, f32 = torch.int32, torch.float32
    kw = dict(ws=ws, stream=stream)
    off = dd.dd_select_diagonals(scores, K, offsets_out=new((1, K), i32), **kw)[0]
    out = [off, dd.dd_fwd(X, off, V, N, Y=new((T, N), X.dtype), **kw), dd.dd_bwd_input(dY, off, V, M, dX=new((T, M), X.dtype), **kw),
           dd.dd_bwd_weight(X, dY, off, dValues=new((K, L), f32), **kw),
           *dd.dd_bwd(X, dY, off, V, dX=new((T, M), X.dtype), dValues=new((K, L), f32), **kw)]
    mag = dd.dd_diag_magnitude(V, new((K,), f32), stream=stream)
    out += [mag, *dd.dd_diagheur_update(D, off, mag, scores[0], K // 2, new((K,), i32), new((K,), i32), **kw)]
    if X.dtype == torch.bfloat16 and M % 256 == 0:
        pre = dd.dd_prepare(off, V, M, N)
        off2, pre = dd.dd_select_prepare(scores[0], V, M, N, offsets_out=new((K,), i32), prepared=pre, stream=stream)
        out += [off2, dd.dd_fwd(X, None, None, N, Y=new((T, N), X.dtype), prepared=pre, stream=stream),
                dd.dd_fwd(X, off, None, N, Y=new((T, N), X.dtype), prepared=pre, algo=dd.DD_ALGO_BLOCKS, stream=stream),
                dd.dd_bwd_input(dY, None, None, M, dX=new((T, M), X.dtype), prepared=pre, stream=stream),
                *dd.dd_bwd(X, dY, off, None, dX=new((T, M), X.dtype), dValues=new((K, L), f32), prepared=pre, **kw)]
    return out


@pytest.mark.parametrize("dtype", [torch.float32, torch.bfloat16])
@pytest.mark.parametrize("T,M,N,K", [(0, 64, 128, 4), (1, 64, 64, 8), (200, 256, 512, 51), (300, 768, 256, 20)])
def test_both_ways_agree(monkeypatch, T, M, N, K, dtype):
    if T == 0 and dtype == torch.bfloat16:
        pytest.skip("one type is enough for no tokens")
    args = _layer(T, M, N, K, dtype)
    ws = dd.Workspace()
    ws.get(1 << 26, args[0].device)
    stream = torch.cuda.Stream()
    short = _calls(*args, ws)
    torch.cuda.synchronize()
    with torch.cuda.stream(stream):  # what the calls need is filled there too
        with_stream = _calls(*args, ws, stream)
    torch.cuda.synchronize()
    allocated = _calls(*args, ws, given=False)
    torch.cuda.synchronize()
    with monkeypatch.context() as m:
        m.setattr(binding, "_fast", _Declines())
        long = _calls(*args, dd.Workspace())
    torch.cuda.synchronize()
    assert len(short) == len(long) == len(with_stream) == len(allocated)
    for a, *others in zip(short, long, with_stream, allocated):
        assert all(torch.equal(a, b) and a.dtype == b.dtype and a.shape == b.shape for b in others)


def test_only_plain_calls_are_answered():
    X, dY, V, _ = _layer(16, 64, 64, 8, torch.float32)
    off, Y = torch.arange(8, dtype=torch.int32, device="cuda"), torch.empty_like(dY)
    plain = dict(src=X, off=off, V=V, Y=Y, N=64, algo=0, ws=None)
    say = lambda **k: binding._fast.product(0, *{**plain, **k}.values(), None)
    assert say() is Y
    new = say(Y=None)
    assert type(new) is torch.Tensor and torch.equal(new, Y) and not new.requires_grad
    sub = X.as_subclass(type("Sub", (torch.Tensor,), {}))
    for change in (dict(Y=Y[:8]), dict(Y=Y.T.contiguous().T), dict(Y=Y.bfloat16()), dict(src=sub), dict(src=X.cpu()), dict(src=X.double()),
                   dict(src=X[0]), dict(src=X[:, :32]), dict(off=off.long()), dict(off=off[::2]), dict(V=V[:4]), dict(V=None), dict(N=63), dict(N=64.0),
                   dict(N=0), dict(algo=True), dict(algo=-1), dict(ws=()), dict(ws=X), dict(src=3)):
        assert say(**change) is None, change
    # a block that is too small is grown by the long way
    Xw, dYw, Vw, _ = _layer(300, 768, 256, 20, torch.bfloat16)
    ws, offw = dd.Workspace(), torch.arange(20, dtype=torch.int32, device="cuda")
    need = dd.dd_workspace_bytes(dd.DD_OP_BWD, dd.make_layer(300, 768, 256, 20, torch.bfloat16))
    ws.get(need - 1, Xw.device)
    dd.dd_bwd(Xw, dYw, offw, Vw, dX=torch.empty_like(Xw), dValues=torch.empty((20, 256), device="cuda"), ws=ws)
    assert need > 1 and ws.buf.numel() >= need
    # what the library refuses is raised from the short way too
    with pytest.raises(dd.DynaDiagError):
        dd.dd_fwd(X, off, V, 64, Y=Y, algo=77)
    torch.cuda.synchronize()


def test_wrapped_tensors_take_the_long_way():
    X, dY, V, _ = _layer(16, 64, 64, 8, torch.float32)
    off, seen = torch.arange(8, dtype=torch.int32, device="cuda"), []

    def f(x):
        seen.append(binding._fast.product(0, x, off, V, torch.empty_like(dY), 64, 0, None, None))
        return x
    torch.func.vmap(f)(X[None])
    torch.func.grad(lambda x: f(x).sum())(X)
    assert seen == [None, None]


def test_an_interrupt_is_not_lost():
    X, dY, V, _ = _layer(16, 64, 64, 8, torch.float32)
    off = torch.arange(8, dtype=torch.int32, device="cuda")

    class Interrupted:
        asked = 0

        @property
        def cuda_stream(self):
            self.asked += 1
            if self.asked == 1:
                raise KeyboardInterrupt
            return torch.cuda.current_stream().cuda_stream

    with pytest.raises(KeyboardInterrupt):
        dd.dd_fwd(X, off, V, 64, Y=torch.empty_like(dY), stream=Interrupted())
