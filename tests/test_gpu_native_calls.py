"""The native part of the binding against its long way: a call with an explicit stream always goes the long way, so every
entry point is called both ways on the same inputs and has to give the same bits, with and without the caller's
buffers; what the native part does not take has to work, or fail, as it does on the long way."""
import ctypes
import threading

import numpy as np
import pytest

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def gpu():
    import torch

    if not torch.cuda.is_available():
        pytest.skip("no GPU")
    from paper_1610_06209_amd import binding

    class G:
        pass

    g = G()
    g.torch, g.b, g.dev = torch, binding, torch.device("cuda:0")
    return g


def _inputs(g, n=1024, batch=37, L=3, seed=1):
    t = g.torch
    gen = t.Generator(device=g.dev)
    gen.manual_seed(seed)
    x = t.randn((batch, n), generator=gen, device=g.dev)
    d = t.randint(0, 2, (L, 3, n), generator=gen, device=g.dev).float() * 2 - 1
    return x, d


def _calls(g, n=1024):
    """name -> (function of the keyword arguments left open, keyword of the result buffer)"""
    t, b = g.torch, g.b
    x, d = _inputs(g, n)
    d1, d2, d3 = d[0]
    words = b.spinner_pack_signs(d)
    codes = b.spinner_sign_codes(x, d1, d2, d3, 512)
    y, saved = b.spinner_layer_forward(x, d1, d2, d3, 0.5)
    spectrum = b.spinner_struct_prepare("toeplitz", t.randn(2 * n - 1, device=g.dev), n)
    A, w = t.randn((n, 44), device=g.dev), t.rand(n, device=g.dev)
    return {
        "apply": (lambda **k: b.spinner_apply(x, d1, d2, d3, 100, "none", 2, **k), "out"),
        "apply features": (lambda **k: b.spinner_apply(x, d1, d2, d3, None, 1, 2.5, **k), "out"),
        "apply_signs": (lambda **k: b.spinner_apply_signs(x, words, triple=2, **k), "out"),
        "apply_blocks": (lambda **k: b.spinner_apply_blocks(x, d, 512, "cossin", 3.0, **k), "out"),
        "hash": (lambda **k: b.spinner_hash(x, d, **k), "out_idx"),
        "hash_signs": (lambda **k: b.spinner_hash_signs(x, words, 2, **k), "out_idx"),
        "sign_codes": (lambda **k: b.spinner_sign_codes(x, d1, d2, d3, 256, **k), "codes"),
        "sign_codes_signs": (lambda **k: b.spinner_sign_codes_signs(x, words, triple=1, **k), "codes"),
        "angular_gram": (lambda **k: b.spinner_angular_gram(codes, codes[:5], 512, **k), "out"),
        "layer_forward": (lambda **k: b.spinner_layer_forward(x, d1, d2, d3, 0.5, **k), "y"),
        "layer_backward": (lambda **k: b.spinner_layer_backward(y, x, saved, d1, d2, d3, 0.5, **k), "dx"),
        "sketch": (lambda **k: b.spinner_sketch(A, w, d1, d2, d3, 128, 1.5, **k), "out"),
        "sketch unweighted": (lambda **k: b.spinner_sketch(A, None, d1, d2, d3, 128, **k), "out"),
        "sketch_gram": (lambda **k: b.spinner_sketch_gram(A, **k), "out"),
        "struct": (lambda **k: b.spinner_struct_apply_ws(x, "toeplitz", spectrum, d1, d2, 1000, 0.5, **k), "out"),
        "struct, kind as a number": (lambda **k: b.spinner_struct_apply_ws(x, 2, spectrum, d1, d2, **k), "out"),
    }


class _Recorder:
    """binding._native with a note of who answered: True for a result, False for None (the long way)."""

    def __init__(self, native):
        self._native, self.served = native, []

    def __getattr__(self, name):
        def call(*args):
            r = getattr(self._native, name)(*args)
            self.served.append(r is not None)
            return r

        return call


@pytest.fixture
def served(gpu, monkeypatch):
    rec = _Recorder(gpu.b._native)
    monkeypatch.setattr(gpu.b, "_native", rec)
    return rec.served


def _all(r):
    return r if isinstance(r, tuple) else (r,)


def test_native_calls_give_the_bits_of_the_long_way(gpu, served):
    t = gpu.torch
    calls = _calls(gpu)
    for name, (f, buffer) in calls.items():
        served.clear()
        long_way = _all(f(stream=t.cuda.current_stream()))
        native = _all(f())
        for p, q in zip(native, long_way):
            assert p.shape == q.shape and p.dtype == q.dtype and t.equal(p, q), name
        mine = t.zeros_like(native[0])
        back = _all(f(**{buffer: mine}))
        assert back[0] is mine and t.equal(mine, long_way[0]), name
        assert served == [False, True, True], name
    assert {name.split()[0].split(",")[0] for name in calls} == {m.replace("struct_apply_ws", "struct") for m in dir(gpu.b._native._native) if m[0] != "_"}


def test_native_calls_with_a_workspace(gpu, served):
    t, b = gpu.torch, gpu.b
    x, d = _inputs(gpu, 1 << 17, 3, 1)
    need = b.spinner_workspace_bytes(1 << 17, 3, 100, "none")
    assert need
    want = b.spinner_apply(x, *d[0], 100, stream=t.cuda.current_stream())
    assert t.equal(b.spinner_apply(x, *d[0], 100), want)
    assert t.equal(b.spinner_apply(x, *d[0], 100, workspace=t.empty(need, dtype=t.uint8, device=gpu.dev)), want)
    assert served == [False, True, True]
    with pytest.raises(ValueError, match="workspace too small"):
        b.spinner_apply(x, *d[0], 100, workspace=t.empty(need - 1, dtype=t.uint8, device=gpu.dev))


def test_calls_that_the_native_part_leaves_to_the_long_way(gpu, served):
    t, b = gpu.torch, gpu.b
    x, d = _inputs(gpu)
    d1, d2, d3 = d[0]
    words = b.spinner_pack_signs(d)
    want = b.spinner_apply(x, d1, d2, d3, 100, "none", 2.0)
    assert served == [True]
    served.clear()
    # numbers that are no plain Python numbers, a subclass of the tensor, sign words of another type
    assert t.equal(b.spinner_apply(x, d1, d2, d3, np.int64(100), "none", np.float32(2.0)), want)
    assert served == [False]
    # (a parameter is a plain tensor)
    assert t.equal(b.spinner_apply(t.nn.Parameter(x), d1, d2, d3, 100, "none", 2.0), want)
    assert served == [False, True]
    served.clear()

    class Sub(t.Tensor):
        pass

    assert t.equal(b.spinner_apply(x.as_subclass(Sub), d1, d2, d3, 100, "none", 2.0).as_subclass(t.Tensor), want)
    with pytest.raises(ValueError, match="contiguous"):
        b.spinner_apply(x.t(), d1, d2, d3)
    with pytest.raises(ValueError, match="contiguous"):
        b.spinner_hash_signs(x.double(), words, 1)
    with pytest.raises(ValueError, match="contiguous"):
        b.spinner_layer_forward(x.cpu(), d1, d2, d3)
    with pytest.raises(ValueError, match="diagonal length"):
        b.spinner_apply(x, d1[:512], d2, d3)
    with pytest.raises(ValueError, match="wrong size"):
        b.spinner_apply(x, d1, d2, d3, 100, out=t.empty(5, device=gpu.dev))
    with pytest.raises(ValueError, match="too small"):
        b.spinner_apply_signs(x, words, triple=3)
    with pytest.raises(KeyError):
        b.spinner_apply(x, d1, d2, d3, 100, "tanh")
    for m in (0, -1, 1025):
        with pytest.raises((b.SpinnerError, RuntimeError)):
            b.spinner_apply(x, d1, d2, d3, m)
    bad = x[:, :1000].contiguous()
    with pytest.raises(b.SpinnerError) as e:
        b.spinner_layer_forward(bad, d1[:1000].contiguous(), d2[:1000].contiguous(), d3[:1000].contiguous())
    assert e.value.status == b.SPINNER_ERR_BAD_N
    with pytest.raises(b.SpinnerError) as e:          # 4 bytes past a 16-byte boundary
        b.spinner_apply(x.flatten()[1:1025].reshape(1, 1024), d1, d2, d3)
    assert e.value.status == b.SPINNER_ERR_ALIGNMENT
    # a host tensor or a shorter diagonal where the kernels cannot tell
    for f in (lambda: b.spinner_apply_signs(x, words.cpu()), lambda: b.spinner_apply_signs(x, words, triple=-1),
              lambda: b.spinner_layer_forward(x, d1[:512], d2, d3), lambda: b.spinner_sign_codes(x, d1, d2, d3[:1020])):
        with pytest.raises(ValueError):
            f()
    # the wrong type of tensor where only a wrapped one can tell: no data pointer to take
    with pytest.raises(RuntimeError):
        t.func.vmap(lambda v: b.spinner_apply(v, d1, d2, d3))(x.reshape(1, 37, 1024))
    assert len(served) >= 13 and not any(served)
    empty = b.spinner_apply(x[:0], d1, d2, d3, 100)
    assert tuple(empty.shape) == (0, 100)


def test_an_error_of_hip_is_raised_and_the_call_not_made_again(gpu):
    # an error that an earlier HIP call left behind is met by the check behind the first launch: the kernel is on its way by
    # then, and a second call on the same buffers would transform x twice.  hipSetDevice refuses a device that is not there.
    t, b = gpu.torch, gpu.b
    x, d = _inputs(gpu)
    want = b.spinner_apply(x, *d[0])
    t.cuda.synchronize()
    with open("/proc/self/maps") as f:
        hip = ctypes.CDLL(next(w[-1] for w in (line.split() for line in f) if "libamdhip64" in w[-1]))
    native, calls = b._native, []

    class Counting:
        @staticmethod
        def apply(*a):
            calls.append(a)
            return native.apply(*a)

    for i in range(2):
        here = x.clone()
        t.cuda.synchronize()
        if i == 1:
            b._native = Counting
        try:
            assert hip.hipSetDevice(1 << 20) != 0
            with pytest.raises(b.SpinnerError) as e:
                b.spinner_apply(here, *d[0], out=here, stream=None if i else t.cuda.current_stream())
        finally:
            b._native = native
        assert e.value.status == b.SPINNER_ERR_HIP
        t.cuda.synchronize()
        assert t.equal(here, want)
    assert len(calls) == 1
    assert t.equal(b.spinner_apply(x, *d[0]), want)


def test_native_calls_on_side_streams_of_several_threads(gpu, served):
    # every thread on a stream of its own that first waits for a long copy: a call on any other stream would read x too early
    t, b = gpu.torch, gpu.b
    x, d = _inputs(gpu, 1024, 4096)
    words = b.spinner_pack_signs(d)
    want = b.spinner_apply_signs(x, words)
    big = t.empty(1 << 26, device=gpu.dev)
    t.cuda.synchronize()
    got = [None] * 4

    def work(i):
        s = t.cuda.Stream()
        with t.cuda.stream(s):
            for _ in range(20):
                big2 = big.clone()
                late = t.zeros_like(x)
                late.copy_(x)
                got[i] = b.spinner_apply_signs(late, words)
            del big2
        s.synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    for th in threads:
        th.start()
    for th in threads:
        th.join()
    for r in got:
        assert t.equal(r, want)
    assert len(served) == 81 and all(served)
