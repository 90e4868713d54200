"""The compiled marshalling of the binding takes what is plainly right and leaves everything else to Python: either way
the results, and what is refused, are the same."""
import sys
import threading
import time

import pytest
import torch

import paper_2511_04214_amd as brq

BF16, F32 = torch.bfloat16, torch.float32


class Named(torch.Tensor):
    pass


def test_leaves_to_python_what_is_not_on_a_gpu():
    brq.lib()
    n, x, c = brq._native, torch.zeros((4, 512)), torch.zeros(4096, dtype=torch.uint8)
    assert n.rotate_quantize(x, 32, c, c, "tiled", None) is None
    assert n.swiglu_rotate_quantize(x, x, 32, F32, c, c, "tiled", None) is None
    assert n.matrix_rotate_quantize(x, torch.eye(32), c, c, "tiled") is None
    assert n.gemm(c, c, c, c, F32, None, "tiled", "tiled", 4, 4, 512) is None
    assert n.rotate_quantize_gemm(x, 32, c, c, 4, F32, None, "tiled", None) is None
    for f in (n.rotate_quantize, n.swiglu_rotate_quantize, n.matrix_rotate_quantize, n.gemm, n.rotate_quantize_gemm):
        assert f() is None and f(None) is None
    with pytest.raises(TypeError):
        n.bind(1)
    with pytest.raises(ValueError):
        n.bind(0, 0, 0, 0, 0)
    with pytest.raises(ValueError, match="GPU tensor"):
        brq.rotate_quantize_fused(x, 32, codes=c, scales=c, layout="tiled")


@pytest.mark.parametrize("why", ["not built", "another torch"])
def test_the_library_does_without_the_compiled_part(why, monkeypatch):
    brq.lib()
    monkeypatch.setattr(brq, "_lib", None)
    monkeypatch.setattr(brq, "_native", None)
    if why == "not built":
        monkeypatch.delattr(brq, "_binding", raising=False)
        monkeypatch.setitem(sys.modules, brq.__name__ + "._binding", None)
    else:
        monkeypatch.setattr(torch, "__version__", "0.1")
    with pytest.warns(RuntimeWarning, match="compiled part"):
        brq.lib()
    assert brq._native is None and brq.operand_bytes(64, 512) == (16384, 1024)
    x, c = torch.zeros((4, 512)), torch.zeros(4096, dtype=torch.uint8)
    for call in (lambda: brq.rotate_quantize_fused(x, 32, c, c, layout="tiled"), lambda: brq.swiglu_rotate_quantize_fused(x, x, 32, F32, c, c),
                 lambda: brq.matrix_rotate_quantize_fused(x, torch.eye(32), c, c), lambda: brq.mxfp4_gemm(c, c, c, c),
                 lambda: brq.rotate_quantize_gemm_fused(x, 32, c, c, 4)):
        with pytest.raises(ValueError, match="GPU tensor"):
            call()


def bufs(M, K, layout):
    nc, ns = brq.operand_bytes(M, K, layout)
    shapes = ((M, K // 2), (M, K // 32)) if layout == "rowmajor" else ((nc,), (ns,))
    return [torch.zeros(s, dtype=torch.uint8, device="cuda") for s in shapes]


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["rowmajor", "tiled"])
@pytest.mark.parametrize("dtype", [F32, BF16])
def test_both_ways_agree(layout, dtype):
    """A Stream argument takes the way through Python."""
    s = torch.cuda.current_stream()
    g = torch.Generator(device="cuda").manual_seed(1)
    M, N, K = 5, 130, 512
    x = torch.randn((M, 2 * K), generator=g, device="cuda").to(dtype)
    signs = (torch.randint(0, 2, (K,), generator=g, device="cuda") * 2 - 1).to(torch.int8)
    R = torch.linalg.qr(torch.randn((K // 32, 32, 32), generator=g, device="cuda"))[0].contiguous()
    gate, up = x[:, :K], x[:, K:]
    w = brq.rotate_quantize_fused(torch.randn((N, K), generator=g, device="cuda"), 32, layout=layout)
    n = brq._native
    a, b = bufs(M, K, layout), bufs(M, K, layout)
    for native, call in (
            (lambda c: n.rotate_quantize(gate, 32, *c, layout, signs), lambda c, **k: brq.rotate_quantize_fused(gate, 32, *c, layout=layout, signs=signs, **k)),
            (lambda c: n.swiglu_rotate_quantize(gate, up, 64, BF16, *c, layout, None), lambda c, **k: brq.swiglu_rotate_quantize_fused(gate, up, 64, BF16, *c, layout=layout, **k)),
            (lambda c: n.matrix_rotate_quantize(gate, R, *c, layout), lambda c, **k: brq.matrix_rotate_quantize_fused(gate, R, *c, layout=layout, **k)),
            (lambda c: n.matrix_rotate_quantize(gate, R[0], *c, layout), lambda c, **k: brq.matrix_rotate_quantize_fused(gate, R[0], *c, layout=layout, **k))):
        for t in a + b:
            t.fill_(9)
        assert native(a) == 0
        got = call(b, stream=s)
        assert got[0] is b[0] and got[1] is b[1] and all(torch.equal(p, q) for p, q in zip(a, b))
        got = call(a)
        assert got[0] is a[0] and got[1] is a[1] and all(torch.equal(p, q) for p, q in zip(a, b))
    sizes = dict(M=M, N=N, K=K) if layout == "tiled" else {}
    for out_dtype in (F32, BF16):
        y = n.gemm(*a, *w, out_dtype, None, layout, layout, *(sizes.get(k) for k in "MNK"))
        want = brq.mxfp4_gemm(*a, *w, out_dtype=out_dtype, a_layout=layout, w_layout=layout, stream=s, **sizes)
        assert y.dtype == out_dtype and y.device == want.device and not y.requires_grad and torch.equal(y, want)
        out = torch.zeros((M, N + 6), dtype=out_dtype, device="cuda")[:, :N]
        assert brq.mxfp4_gemm(*a, *w, out=out, a_layout=layout, w_layout=layout, **sizes) is out and torch.equal(out, want)
        z = n.rotate_quantize_gemm(gate, 32, *w, N, out_dtype, None, layout, None)
        assert torch.equal(z, brq.rotate_quantize_gemm_fused(gate, 32, *w, N, out_dtype=out_dtype, w_layout=layout, stream=s))


@pytest.mark.gpu
def test_what_is_refused_stays_refused():
    M, N, K = 4, 64, 512
    x = torch.randn((M, K), device="cuda")
    c, s = bufs(M, K, "rowmajor")
    w = brq.rotate_quantize_fused(torch.randn((N, K), device="cuda"), 32)
    q = brq.rotate_quantize_fused
    for error, call in (
            (ValueError, lambda: q(x.t(), 32, c, s)), (ValueError, lambda: q(x, 32, c[:2], s)), (ValueError, lambda: q(x, 32, c.to(torch.int8), s)),
            (TypeError, lambda: q(x.half(), 32, c, s)), (ValueError, lambda: q(x, 32, c, s, layout="columns")),
            (ValueError, lambda: q(x, 32, c, s, signs=torch.ones(K, device="cuda"))),
            (ValueError, lambda: brq.mxfp4_gemm(c, s, *w, M=M + 1)), (ValueError, lambda: brq.mxfp4_gemm(c, s[:, :-1].contiguous(), *w)),
            (ValueError, lambda: brq.mxfp4_gemm(c, s, w[0].flatten(), w[1].flatten())), (TypeError, lambda: brq.mxfp4_gemm(c, s, *w, out_dtype=torch.float16)),
            (ValueError, lambda: brq.mxfp4_gemm(c, s, *w, out=torch.zeros((M, N + 1), device="cuda"))),
            (ValueError, lambda: brq.rotate_quantize_gemm_fused(x, 32, w[0][:-1], w[1][:-1], N))):
        with pytest.raises(error):
            call()
    for status, call in ((3, lambda: q(x, 48, c, s)), (4, lambda: q(x.flatten()[1:].as_strided((M - 1, K), (K, 1)), 32, c, s)),
                         (3, lambda: brq.rotate_quantize_gemm_fused(x, 64, *w, N)), (2, lambda: brq.rotate_quantize_gemm_fused(x.repeat(5, 1), 32, *w, N))):
        with pytest.raises(brq.BrqError) as e:
            call()
        assert e.value.status == status
    # taken, by the way through Python
    n = x.as_subclass(Named)
    assert brq._native.rotate_quantize(n, 32, c, s, "rowmajor", None) is None
    q(x, 32, c, s)
    want = c.clone()
    c.zero_()
    q(n, 32, c, s)
    assert torch.equal(c, want)
    assert brq._native.rotate_quantize(torch.nn.Parameter(x), 32, c, s, "rowmajor", None) == 0
    assert brq.mxfp4_gemm(c[:0], s[:0], *w).shape == (0, N)
    with torch.cuda.stream(torch.cuda.Stream()):
        c.zero_()
        q(x, 32, c, s)
        torch.cuda.current_stream().synchronize()
    assert torch.equal(c, want)


@pytest.mark.gpu
def test_other_threads_run_while_the_result_is_allocated():
    """A result that fits only once the allocator has given memory back to the driver, which waits for the GPU's work: as on the
    way through Python, where torch.empty lets go of the interpreter's lock, another thread must not stand still for it."""
    M = N = 12288
    a = brq.rotate_quantize_fused(torch.randn((M, 512), device="cuda"), 32)
    busy, sink = torch.randn((8192, 8192), device="cuda"), torch.empty((8192, 8192), device="cuda")
    torch.mm(busy, busy, out=sink)

    def longest_pause(**kw):
        """of another thread, and how long the call took, in seconds"""
        torch.cuda.synchronize()
        torch.cuda.empty_cache()
        torch.cuda.set_per_process_memory_fraction((torch.cuda.memory_reserved() + (800 << 20)) / torch.cuda.get_device_properties(0).total_memory)
        try:
            held = torch.empty((512 << 20,), dtype=torch.uint8, device="cuda")
            del held                                                    # 512 MB in the allocator's hands; the result is 576 MB
            pause, done = [0.0], threading.Event()

            def ticks():
                last = time.perf_counter()
                while not done.is_set():
                    time.sleep(0.001)
                    now = time.perf_counter()
                    pause[0], last = max(pause[0], now - last), now

            t = threading.Thread(target=ticks)
            t.start()
            for _ in range(60):
                torch.mm(busy, busy, out=sink)
            start = time.perf_counter()
            y = brq.mxfp4_gemm(*a, *a, **kw)
            took = time.perf_counter() - start
            done.set()
            t.join()
            return pause[0], took, y
        finally:
            torch.cuda.set_per_process_memory_fraction(1.0)

    pause, took, want = longest_pause(stream=torch.cuda.current_stream())       # the way through Python
    print("through Python: call %.3f s, pause %.3f s" % (took, pause))
    assert took > 0.1 and pause < took / 2, "the allocation did not wait: this measures nothing"
    want = want.cpu()
    pause, took, y = longest_pause()
    print("compiled: call %.3f s, pause %.3f s" % (took, pause))
    assert took > 0.1 and pause < took / 2
    assert torch.equal(y.cpu(), want)


class Layer:
    """The five calls on buffers of their own, without a stream argument: the compiled way."""

    def __init__(self, seed, M=5, N=130, K=512, layout="tiled"):
        g = torch.Generator(device="cuda").manual_seed(seed)
        self.M, self.N, self.K, self.layout = M, N, K, layout
        self.x = torch.randn((M, 2 * K), generator=g, device="cuda").to(BF16)
        self.R = torch.linalg.qr(torch.randn((K // 32, 32, 32), generator=g, device="cuda"))[0].contiguous()
        self.w = brq.rotate_quantize_fused(torch.randn((N, K), generator=g, device="cuda"), 32, layout=layout)
        self.q = [bufs(M, K, layout) for _ in range(3)]
        self.y = torch.zeros((M, N), device="cuda")

    def clear(self):
        for t in [t for q in self.q for t in q] + [self.y]:
            t.zero_()

    def natively(self):
        """(what each call of the compiled part answers)"""
        n, lay, size = brq._native, self.layout, (self.M, self.N, self.K)
        gate, up = self.x[:, :self.K], self.x[:, self.K:]
        return [n.rotate_quantize(gate, 32, *self.q[0], lay, None), n.swiglu_rotate_quantize(gate, up, 32, BF16, *self.q[1], lay, None),
                n.matrix_rotate_quantize(gate, self.R, *self.q[2], lay), n.gemm(*self.q[1], *self.w, BF16, None, lay, lay, *size),
                n.rotate_quantize_gemm(gate, 32, *self.w, self.N, F32, self.y, lay, None)]

    def step(self, **kw):
        gate, up, lay = self.x[:, :self.K], self.x[:, self.K:], self.layout
        brq.rotate_quantize_fused(gate, 32, *self.q[0], layout=lay, **kw)
        brq.swiglu_rotate_quantize_fused(gate, up, 32, BF16, *self.q[1], layout=lay, **kw)
        brq.matrix_rotate_quantize_fused(gate, self.R, *self.q[2], layout=lay, **kw)
        z = brq.mxfp4_gemm(*self.q[1], *self.w, out_dtype=BF16, a_layout=lay, w_layout=lay, M=self.M, N=self.N, K=self.K, **kw)
        brq.rotate_quantize_gemm_fused(gate, 32, *self.w, self.N, out=self.y, w_layout=lay, **kw)
        return [t for q in self.q for t in q] + [self.y, z]


def same(got, want):
    return len(got) == len(want) and all(torch.equal(a, b) for a, b in zip(got, want))


def keep_busy():
    """About 0.2 s of work on the current stream."""
    a = torch.randn((8192, 8192), device="cuda")
    out = torch.empty_like(a)
    for _ in range(30):
        torch.mm(a, a, out=out)
    return torch.cuda.current_stream().record_event()


@pytest.mark.gpu
def test_calls_go_to_the_current_stream():
    """The default stream is busy: a call that went there would be late for the copies made on the side stream."""
    layer, side = Layer(21), torch.cuda.Stream()
    want = [t.cpu() for t in layer.step(stream=torch.cuda.current_stream())]
    with torch.cuda.stream(side):
        torch.empty((1 << 20,), device="cuda")           # (the side stream's result is not the first thing allocated there)
    layer.clear()
    torch.cuda.synchronize()
    late = keep_busy()
    with torch.cuda.stream(side):
        got = [t.cpu() for t in layer.step()]
    assert not late.query(), "the default stream was not busy long enough: this shows nothing"
    assert same(got, want)
    torch.cuda.synchronize()


@pytest.mark.gpu
@pytest.mark.parametrize("layout", ["rowmajor", "tiled"])
def test_calls_without_a_stream_in_a_hip_graph(layout):
    layer = Layer(22, layout=layout)
    xs = [layer.x.clone(), layer.x.flip(0).contiguous(), layer.x * 3]
    eager = []
    for x in xs:
        layer.x.copy_(x)
        eager.append([t.clone() for t in layer.step()])
    graph = torch.cuda.CUDAGraph()
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        out = layer.step()
    for _ in range(2):
        for x, want in zip(xs, eager):
            layer.x.copy_(x)
            layer.clear()
            graph.replay()
            torch.cuda.synchronize()
            assert same(out, want)
            assert same(layer.step(), want)                  # eager work between the replays


class Watching(torch.overrides.TorchFunctionMode):
    def __init__(self):
        super().__init__()
        self.seen = 0

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.seen += 1
        return func(*args, **(kwargs or {}))


@pytest.mark.gpu
def test_watched_and_batched_tensors_are_left_to_python():
    layer = Layer(23)
    want = [t.clone() for t in layer.step()]
    layer.clear()
    with Watching() as mode:
        assert layer.natively() == [None] * 5
        before = mode.seen
        got = layer.step()
        assert mode.seen > before, "the mode saw nothing of the calls"
    assert same(got, want)
    answers = layer.natively()
    assert answers[:3] == [0, 0, 0] and torch.equal(answers[3], want[-1]) and answers[4] is layer.y

    def batched(x):
        layer.x = x
        assert layer.natively()[:3] == [None] * 3 and layer.natively()[4] is None
        for kw in ({}, dict(stream=torch.cuda.current_stream())):
            with pytest.raises(RuntimeError):
                layer.step(**kw)                             # no memory of its own: refused by both ways
        return x

    torch.vmap(batched)(torch.stack([layer.x, layer.x]))


@pytest.mark.gpu
def test_threads_with_streams_of_their_own():
    layers = [Layer(30 + i, M=3 + i) for i in range(4)]
    wants = [[t.cpu() for t in layer.step()] for layer in layers]
    wrong = []

    def work(layer, want):
        try:
            with torch.cuda.stream(torch.cuda.Stream()):
                for i in range(20):
                    layer.clear()
                    if not same([t.cpu() for t in layer.step()], want):
                        wrong.append((layer.M, i))
        except Exception as e:
            wrong.append(e)

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=a) for a in zip(layers, wants)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not wrong
