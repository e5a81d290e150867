"""The extension behind runner.py's methods (py_calls.cpp): it takes a call whose arguments are all as they should be, and leaves every
other one to the Python code."""
import numpy as np
import pytest
import torch

from paper_2511_20426_amd import binding as B

SHAPE = (2, 128, 60, 0, 0)


def test_calls_that_are_not_taken():
    x, w = torch.zeros(4, 128, dtype=torch.bfloat16), torch.zeros(8, 128, dtype=torch.bfloat16)
    q = torch.zeros(60, 2, 128, dtype=torch.bfloat16)
    for a in ((x, w, None), (1, 2, 3), (x, w), (None, w, None), (x, w, 5)):      # host tensors, no tensors, too few
        assert B.calls.linear(*a) is None
    assert B.calls.rope(1, SHAPE, q, 0, None) is None and B.calls.rope(0, SHAPE, q, 0, None) is None
    assert B.calls.forward(1, SHAPE, q, [0], 0, None, None) is None and B.calls.forward(1, SHAPE, q, [0], 0, None, (0, 1, 2)) is None
    assert B.calls.forward_rope(1, SHAPE, q, range(1), 0, None) is None
    assert B.calls.append_batch(1, SHAPE, [0], [0], 0, [q], [q]) is None
    assert B.calls.append_batch(1, SHAPE[:4], [0], [0], 0, [q], [q]) is None and B.calls.append_batch(1, list(SHAPE), [0], [0], 0, [q], [q]) is None
    assert B.calls.qkv_publish(1, SHAPE, x, w, [0], [0], 0, None) is None
    for bad in ((1, 2), (0,) * 7, (1.0,) * 7, (np.int64(5),) * 7):
        with pytest.raises(TypeError):
            B.calls.bind(*bad)


def _pool():
    from paper_2511_20426_amd.runner import CascadePool
    return CascadePool(heads=2, head_dim=128, frames_per_block=3, grid_h=4, grid_w=5, rope_dims=(44, 42, 42), rope_theta=10000.0, sink_blocks=0,
                       window_blocks=2, max_inflight=3, page_tokens=128, dtype="bf16")


class _Sub(torch.Tensor):
    pass


@pytest.mark.gpu
def test_both_ways_do_the_same():
    """The same calls taken by the extension and, for one argument of another kind each, by the Python code: same results, same pages."""
    from paper_2511_20426_amd.runner import linear
    g = torch.Generator(device="cuda:0").manual_seed(3)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda:0").to(torch.bfloat16)  # noqa: E731
    k, v, q = [rand(60, 2, 128) for _ in range(2)], [rand(60, 2, 128) for _ in range(2)], rand(120, 2, 128)
    x, w = rand(33, 256), rand(24, 256)
    wq, xq = rand(768, 256), rand(120, 256)
    out = {}
    for fast in (True, False):
        p = _pool()
        p.pool.fill_(0xAB)
        num = int if fast else np.int64
        ten = (lambda t: t) if fast else (lambda t: t.as_subclass(_Sub))
        assert p.append_batch([num(0), num(1)], (250, 500), 0, k, tuple(v)) == [0, 1]
        got = [p.rope(ten(q), 3), p.forward_rope(ten(q), [num(0), 1], B.CA_BLOCK_CAUSAL), p.forward(p.rope(q, 3), (num(0), 1), B.CA_BIDIRECTIONAL),
               p.forward(ten(q[:60]), [0, 1], B.CA_BIDIRECTIONAL, share=(1, 1)), linear(ten(x), w),
               p.qkv_publish(ten(xq), wq, [0, num(1)], [0, 250], 0)]
        y = torch.empty(33, 40, dtype=torch.bfloat16, device="cuda:0")[:, :24]
        assert linear(ten(x), w, out=y) is y
        o = torch.empty_like(q)
        assert p.forward_rope(ten(q), [0, 1], 0, out=o) is o
        torch.cuda.synchronize()
        out[fast] = [t.as_subclass(torch.Tensor).clone() for t in got] + [y.clone(), o, p.pool[:2 * 2 * 65536].clone()]
    for a, b in zip(out[True], out[False]):
        assert torch.equal(a.view(torch.int16) if a.dtype == torch.bfloat16 else a, b.view(torch.int16) if b.dtype == torch.bfloat16 else b)


@pytest.mark.gpu
def test_what_was_refused_is_refused():
    from paper_2511_20426_amd.runner import linear
    p = _pool()
    q = torch.zeros(60, 2, 128, dtype=torch.bfloat16, device="cuda:0")
    with pytest.raises(B.CascadeAttnError):
        p.forward(q, [7], B.CA_BIDIRECTIONAL)                            # not in the cache
    with pytest.raises(B.CascadeAttnError):
        p.append_batch([0, 0], [0, 0], 0, [q, q], [q, q])                # one block twice
    for bad in (q.float(), q[:59], q.cpu(), q.transpose(0, 1), q[:, :1], q.view(60, 256)):
        with pytest.raises((AssertionError, IndexError)):
            p.append_batch([0], [0], 0, [bad], [bad])
        with pytest.raises((AssertionError, IndexError)):
            p.forward_rope(bad, [0], 0)
    x, w = torch.zeros(4, 128, dtype=torch.bfloat16, device="cuda:0"), torch.zeros(8, 128, dtype=torch.bfloat16, device="cuda:0")
    for a in ((x.float(), w), (x, w.t()), (x, w[:, :64]), (x.cpu(), w), (x, w, x)):
        with pytest.raises(AssertionError):
            linear(*a)
    with pytest.raises(B.CascadeAttnError):
        linear(x[:, :64], w[:, :64])                                     # k must be a multiple of 128
    p.ctx.close()
    with pytest.raises(B.CascadeAttnError):
        p.rope(q, 0)


def _outs(like):
    """Results that a launch must not be given: of another type (a larger and a smaller one), in pageable host memory, of another shape."""
    return [torch.empty_like(like, dtype=torch.float32), torch.empty_like(like, dtype=torch.uint8), torch.empty_like(like, device="cpu"),
            torch.empty_like(like[:-1])]


@pytest.mark.gpu
def test_results_of_another_type_or_in_host_memory_are_refused():
    """... before anything is launched, by the extension (which leaves them to the Python code) and by the Python code."""
    from paper_2511_20426_amd.runner import linear
    p = _pool()
    g = torch.Generator(device="cuda:0").manual_seed(4)
    rand = lambda *s: torch.randn(s, generator=g, device="cuda:0").to(torch.bfloat16)  # noqa: E731
    q, x, w, xq, wq = rand(60, 2, 128), rand(33, 256), rand(24, 256), rand(60, 256), rand(768, 256)
    p.append_batch([0], [0], 0, [q], [q])
    calls = ((lambda a, out: p.forward(a, [0], 0, out=out), q), (lambda a, out: p.forward(a, [0], 0, out=out, share=(0, 1)), q),
             (lambda a, out: p.forward(a, [0], 0, out=out, static_scratch=True), q), (lambda a, out: p.forward_rope(a, [0], 0, out=out), q),
             (lambda a, out: p.qkv_publish(a, wq, [0], [0], 0, q_out=out), xq), (lambda a, out: linear(a, w, out=out), x))
    for call, a in calls:
        good = torch.empty((33, 24), dtype=torch.bfloat16, device="cuda:0") if a is x else torch.empty_like(q)
        for as_given in (a, a.as_subclass(_Sub)):
            for out in _outs(good):
                with pytest.raises(AssertionError):
                    call(as_given, out)
            assert call(as_given, good) is good
        # memory that kernels reach, on the host: taken as before
        pinned = torch.empty(good.shape, dtype=good.dtype, pin_memory=True)
        assert call(a, pinned) is pinned
        torch.cuda.synchronize()
        assert torch.equal(pinned.view(torch.int16), good.cpu().view(torch.int16))
    for bad in (wq.cpu(), wq.float()):
        with pytest.raises(AssertionError):
            p.qkv_publish(xq, bad, [0], [0], 0)


@pytest.mark.gpu
def test_streams_and_threads():
    """A call goes to the calling thread's stream of the moment."""
    import threading
    from paper_2511_20426_amd.runner import linear
    x, w = torch.randn(300, 512, device="cuda:0").to(torch.bfloat16), torch.randn(256, 512, device="cuda:0").to(torch.bfloat16)
    want = linear(x, w)
    torch.cuda.synchronize()
    got = {}

    def work(i):
        s = torch.cuda.Stream()
        with torch.cuda.stream(s):
            for _ in range(20):
                busy = x.clone()                                         # ordered on this stream only
                got[i] = linear(busy, w)
        s.synchronize()
    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert len(got) == 4 and all(torch.equal(want, y) for y in got.values())
    # recorded into a graph: the capturing stream is the current one
    y = torch.empty_like(want)
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        linear(x, w, out=y)
    for _ in range(3):
        y.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(y, want)


@pytest.mark.gpu
def test_what_an_allocation_raises_comes_through():
    """An error that a dispatch mode raises inside the extension's torch.empty is the caller's to see."""
    from torch.utils._python_dispatch import TorchDispatchMode

    from paper_2511_20426_amd.runner import linear

    class Refuses(TorchDispatchMode):
        def __torch_dispatch__(self, func, types, args=(), kwargs=None):
            raise ValueError("no memory for you")

    x, w = torch.zeros(4, 128, dtype=torch.bfloat16, device="cuda:0"), torch.zeros(8, 128, dtype=torch.bfloat16, device="cuda:0")
    with Refuses(), pytest.raises(ValueError, match="no memory for you"):
        linear(x, w)
    assert linear(x, w).shape == (4, 8)
