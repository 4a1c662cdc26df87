"""The native module of the Python binding against the ctypes path that it stands in front of: same results where it
answers, and nothing but None where a call is not the plain one (the ctypes path then runs it or raises)."""
import threading

import numpy as np
import pytest

from paper_2509_01229_amd import api

import gpu_helpers as H


class _Nothing:
    """A native module that leaves every call to the ctypes path."""
    gemm = quantize = grouped = staticmethod(lambda *a: None)


def _both(monkeypatch, call):
    """call() through the native module (which has to answer) and through the ctypes path"""
    import torch

    answers, native = [], api._native

    class Watched:
        def __getattr__(self, name):
            def run(*a):
                answers.append(getattr(native, name)(*a))
                return answers[-1]
            return run

    monkeypatch.setattr(api, "_native", Watched())
    fast = call()
    assert answers and all(a is not None for a in answers)
    monkeypatch.setattr(api, "_native", _Nothing)
    general = call()
    monkeypatch.setattr(api, "_native", native)
    flat = lambda r: [t for t in (r if isinstance(r, tuple) else (r,)) if t is not None]
    assert len(flat(fast)) == len(flat(general))
    for f, g in zip(flat(fast), flat(general)):
        assert type(f) is type(g) and f.dtype == g.dtype and f.shape == g.shape and f.device == g.device and f.stride() == g.stride()
        assert torch.equal(f.view(torch.uint8), g.view(torch.uint8))
    return fast


@pytest.mark.gpu
@pytest.mark.parametrize("M,N,K,g", [(1, 64, 256, 64), (9, 2048, 4096, 128), (45, 128, 8192, 64), (300, 320, 768, 64)])
def test_gemm_and_quantisation(monkeypatch, M, N, K, g):
    import torch

    gen = torch.Generator(device="cuda").manual_seed(M)
    W = H.RandomWeights(N, K, g, seed=M)
    X = torch.randn((M, K), generator=gen, device="cuda").half()
    smooth = torch.rand(K, generator=gen, device="cuda") + 0.5
    api.w4a8_gemm(*W.activations(M), W.codes, W.gparams, W.scales, N, K, g)  # (makes this stream's workspace)
    q, s = _both(monkeypatch, lambda: api.w4a8_quantize_activations(X))
    _both(monkeypatch, lambda: api.w4a8_quantize_activations(X, smooth))
    out_q, out_s = torch.empty_like(q), torch.empty_like(s)
    r = _both(monkeypatch, lambda: api.w4a8_quantize_activations(X, smooth, out_q, out_s, stream=torch.cuda.current_stream().cuda_stream))
    assert r[0] is out_q and r[1] is out_s
    args = (q, s, W.codes, W.gparams, W.scales, N, K, g)
    y = _both(monkeypatch, lambda: api.w4a8_gemm(*args))
    ws = torch.zeros(max(16, api.w4a8_gemm_workspace_size(M, N, K, g)), dtype=torch.uint8, device="cuda")
    out = torch.empty_like(y)
    for workspace in (ws, ws[:16]):
        assert _both(monkeypatch, lambda: api.w4a8_gemm(*args, out=out, workspace=workspace)) is out
        assert torch.equal(out, y)


@pytest.mark.gpu
@pytest.mark.parametrize("rows", [[3], [0, 5, 40, 1], [16] * 64])
def test_grouped(monkeypatch, rows):
    import torch

    N, K, g, E = 128, 512, 64, len(rows)
    offs = [0] + [int(v) for v in np.cumsum(rows)]
    W = H.RandomWeights(E * N, K, g, seed=E)
    X, s = W.activations(offs[-1])
    args = (X, s, W.codes, W.gparams, W.scales.view(E, N), N, K, g)
    y, acc = _both(monkeypatch, lambda: api.w4a8_grouped_gemm(offs, *args))
    assert acc is None
    out = torch.empty_like(y)
    assert _both(monkeypatch, lambda: api.w4a8_grouped_gemm(offs, *args, out_y=out))[0] is out
    # other sequences of numbers go to the ctypes path
    for other in (tuple(offs), np.array(offs), torch.tensor(offs)):
        assert torch.equal(api.w4a8_grouped_gemm(other, *args)[0], y)


@pytest.mark.gpu
def test_errors_are_those_of_the_ctypes_path(monkeypatch):
    import torch

    N, K, g = 64, 256, 64
    W = H.RandomWeights(N, K, g, seed=1)
    X, s = W.activations(4)
    f16 = torch.zeros(4 * K + 8, dtype=torch.float16, device="cuda")
    calls = [lambda: api.w4a8_quantize_activations(torch.zeros((4, 12), dtype=torch.float16, device="cuda")),
             lambda: api.w4a8_quantize_activations(f16[1:4 * K + 1].view(4, K)),   # (not aligned)
             lambda: api.w4a8_quantize_activations(f16[:4 * K].view(K, 4).t()),   # (not contiguous)
             lambda: api.w4a8_quantize_activations(f16),
             lambda: api.w4a8_gemm(X, s, W.codes[1:], W.gparams, W.scales, N, K, g),
             lambda: api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, N, K, 32),
             lambda: api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, 2 ** 40, K, g),
             lambda: api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, N, K, g, out=torch.empty((4, N), device="cuda")),
             lambda: api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, N, K, g, workspace=torch.zeros(64, device="cuda")),
             lambda: api.w4a8_gemm(X.cpu(), s, W.codes, W.gparams, W.scales, N, K, g),
             lambda: api.w4a8_grouped_gemm([0, 5, 4], X, s, W.codes, W.gparams, W.scales.view(1, N), N, K, g),
             lambda: api.w4a8_grouped_gemm([1, 4], X, s, W.codes, W.gparams, W.scales.view(1, N), N, K, g)]
    native = api._native
    for i, call in enumerate(calls):
        raised = []
        for module in (native, _Nothing):
            monkeypatch.setattr(api, "_native", module)
            with pytest.raises(Exception) as e:
                call()
            raised.append((e.type, str(e.value)))
        assert raised[0] == raised[1], i
    monkeypatch.setattr(api, "_native", native)
    empty = api.w4a8_gemm(X[:0], s[:0], W.codes, W.gparams, W.scales, N, K, g)
    assert empty.shape == (0, N) and api.w4a8_quantize_activations(torch.empty((0, K), dtype=torch.float16, device="cuda"))[0].shape == (0, K)


@pytest.mark.gpu
def test_threads_with_streams_of_their_own():
    import torch

    N, K, g = 512, 8192, 64
    W = H.RandomWeights(N, K, g, seed=5)
    X, s = W.activations(20)
    want, got = api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, N, K, g), [None] * 4
    torch.cuda.synchronize()

    def work(i):
        with torch.cuda.stream(torch.cuda.Stream()):
            outs = [api.w4a8_gemm(X, s, W.codes, W.gparams, W.scales, N, K, g) for _ in range(50)]
            torch.cuda.current_stream().synchronize()
            got[i] = all(torch.equal(o, want) for o in outs)
            torch.cuda.current_stream().synchronize()

    threads = [threading.Thread(target=work, args=(i,)) for i in range(4)]
    [t.start() for t in threads]
    [t.join() for t in threads]
    assert got == [True] * 4


def test_what_the_native_module_leaves_alone():
    """Without a GPU: tensors of the host, other objects, numbers that are no plain integers, the wrong count."""
    import torch

    api.lib()
    X, s, W = torch.zeros((4, 256), dtype=torch.int8), torch.ones(4), torch.zeros(8192, dtype=torch.uint8)
    for bad in (X, np.zeros((4, 256), np.int8), None, 3, "x", torch.nn.Parameter(torch.zeros(4, 256))):
        assert api._native.gemm(bad, s, W, W, s, 64, 256, 64, None, None, None, {}) is None
        assert api._native.quantize(bad, None, None, None, None) is None
        assert api._native.grouped([0, 4], bad, s, W, W, s, 64, 256, 64, None, None) is None
    for offs in ((0, 4), [0], [0, 2.0], [0, True], [0, 2 ** 70], [0] * 70, []):
        assert api._native.grouped(offs, X, s, W, W, s, 64, 256, 64, None, None) is None
    assert api._native.gemm() is None and api._native.quantize(X) is None and api._native.grouped(1) is None


@pytest.mark.parametrize("what", ["missing", "of another torch"])
def test_without_a_native_module_for_this_torch(monkeypatch, what):
    """Only the calls that would use it notice, and they run on the ctypes path: the host functions need the C library alone."""
    import sys
    import types
    import warnings

    import paper_2509_01229_amd as package

    monkeypatch.setattr(api, "_native", None)
    monkeypatch.setattr(api, "_lib", None)
    monkeypatch.delattr(package, "_binding", raising=False)
    other = types.ModuleType("paper_2509_01229_amd._binding")
    other.built_for = "Python 3.9, torch 1.0"
    monkeypatch.setitem(sys.modules, "paper_2509_01229_amd._binding", None if what == "missing" else other)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        packed, gparams = api.liquidquant_pack_from_i8(np.ones((64, 256), np.int8), 64)
        assert packed.size == 64 * 256 // 2 and api.w4a8_describe_launch(8, 64, 256, 64)[0]
    import torch

    X = torch.zeros((4, 256), dtype=torch.int8)   # (on the host: the ctypes path refuses it)
    with pytest.warns(RuntimeWarning, match="no native module"):
        with pytest.raises(TypeError):
            api.w4a8_gemm(X, torch.ones(4), X, X, torch.ones(64), 64, 256, 64)
    with warnings.catch_warnings():
        warnings.simplefilter("error")
        for call in (lambda: api.w4a8_gemm(X, torch.ones(4), X, X, torch.ones(64), 64, 256, 64), lambda: api.w4a8_quantize_activations(X.half()),
                     lambda: api.w4a8_grouped_gemm([0, 4], X, torch.ones(4), X, X, torch.ones(1, 64), 64, 256, 64)):
            with pytest.raises(TypeError):
                call()


def test_the_built_native_module_is_used():
    api.lib()
    assert api._native.__name__ == "paper_2509_01229_amd._binding" and api._native.built_for == api.native_built_for()
