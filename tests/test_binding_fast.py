"""The native side of the binding serves plain calls with the results of the general one and leaves it all others."""
from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

import paper_2208_04187_amd as pkg
from paper_2208_04187_amd import binding


def test_native_side_is_built_and_leaves_host_tensors_alone():
    fast = binding._load_fast()
    assert fast.__name__.endswith("_fastcall")
    x = torch.zeros(2, 2, 8, 8)
    assert fast.compress(x, 8, 2, 1, False, 4) is None and fast.relu_forward(x) is None and fast.compress_maps([x], 8, 2, [1], False) is None
    assert fast.decompress(x, (2, 2, 8, 8), 8, 2, torch.float32, False, 4) is None and fast.compress() is None
    for call in (lambda: pkg.division_compress(x, 8, 2, 1), lambda: pkg.division_compress_3d(x, 8, 2, 1), lambda: pkg.division_relu_forward(x),
                 lambda: pkg.division_compress_maps([x], 8, 2, [1]), lambda: pkg.division_maxpool_forward(x, 2)):
        with pytest.raises(ValueError):
            call()
    with pytest.raises(ValueError):
        fast.bind([1])


def _loaded_anew(monkeypatch):
    """binding._fast as a fresh process finds it"""
    monkeypatch.setattr(binding, "_fast", None)
    return binding._load_fast()


def test_native_side_is_built_where_it_is_missing(monkeypatch, tmp_path):
    from paper_2208_04187_amd import _build
    built = []
    monkeypatch.setattr(binding, "_FAST_PATH", tmp_path / "_fastcall.so")
    monkeypatch.setattr(_build, "build_fastcall", lambda: built.append(True))
    assert _loaded_anew(monkeypatch).__name__.endswith("_fastcall") and built == [True]

    def no_compiler():
        raise RuntimeError("g++ failed")
    monkeypatch.setattr(_build, "build_fastcall", no_compiler)
    with pytest.warns(RuntimeWarning, match="g\\+\\+ failed"):
        assert isinstance(_loaded_anew(monkeypatch), binding._NothingFast)


@pytest.mark.parametrize("entries,version,map_bytes", [(12, 2, None), (12, 1, 104), (11, 1, None), (12, None, None)])
def test_native_side_of_another_library_is_not_used(monkeypatch, entries, version, map_bytes):
    fast = binding._load_fast()
    size = map_bytes or ctypes.sizeof(binding._MapDesc)
    with pytest.raises(ValueError, match="ABI version 1 "):
        fast.bind([1] * entries, version, size)
    bind = fast.bind
    monkeypatch.setattr(fast, "bind", lambda *args: bind([1] * entries, version, size))
    with pytest.warns(RuntimeWarning, match="ABI version 1 "):
        assert isinstance(_loaded_anew(monkeypatch), binding._NothingFast)
    monkeypatch.undo()
    x = torch.zeros(2, 2, 8, 8)
    assert binding._load_fast() is fast and fast.compress(x, 8, 2, 1, False, 4) is None


class _General:
    """The binding without its native side"""

    def __enter__(self):
        binding._load_fast()
        self.fast, binding._fast = binding._fast, binding._NothingFast()

    def __exit__(self, *exc):
        binding._fast = self.fast


def _equal(a, b):
    if isinstance(a, (list, tuple)):
        return type(a) is type(b) and len(a) == len(b) and all(_equal(p, q) for p, q in zip(a, b))
    return a.shape == b.shape and a.dtype == b.dtype and a.device == b.device and torch.equal(a, b)


@pytest.mark.gpu
@pytest.mark.parametrize("dtype,c16", [(torch.float32, False), (torch.bfloat16, False), (torch.float32, True)])
def test_plain_calls_give_what_the_general_ones_give(dtype, c16):
    gen = torch.Generator().manual_seed(3)
    x = torch.randn((3, 5, 14, 14), generator=gen).to(dtype).to("cuda:0")
    v = torch.randn((2, 3, 4, 9, 9), generator=gen).to(dtype).to("cuda:0")
    seed = -(2 ** 63) + 77                                     # negative and beyond 64 bits: seeds count modulo 2^64
    p, q = pkg.division_compress(x, 8, 2, seed, c16=c16), pkg.division_compress_3d(v, 4, 4, 2 ** 64 + 9, c16=c16)
    y, mask = pkg.division_maxpool_forward(x, 3)
    calls = [lambda: pkg.division_compress(x, 8, 2, seed, c16=c16), lambda: pkg.division_compress_3d(v, 4, 4, 2 ** 64 + 9, c16=c16),
             lambda: pkg.division_decompress(p, x.shape, 8, 2, dtype, c16=c16), lambda: pkg.division_decompress(p, list(x.shape), 8, 2, dtype, c16=c16),
             lambda: pkg.division_decompress_3d(q, tuple(v.shape), 4, 4, dtype, c16=c16),
             lambda: pkg.division_compress_maps([x, v], (8, 4), [2, 4], [seed, 2 ** 64 + 9], c16=c16),
             lambda: pkg.division_compress_maps((x, x), 8, 2, (1, 2), c16=c16),
             lambda: pkg.division_decompress_maps([p, q], [x.shape, v.shape], [8, 4], [2, 4], dtype, c16=c16),
             lambda: pkg.division_decompress_maps((p, p), (x.shape, x.shape), 8, 2, [dtype, dtype], c16=c16),
             lambda: pkg.division_relu_forward(x), lambda: pkg.division_relu_compress(x, 8, 2, seed, c16=c16), lambda: pkg.division_dropout_forward(v, 0.25, seed),
             lambda: pkg.division_mask_backward(mask, x), lambda: pkg.division_maxpool_forward(x, 3), lambda: pkg.division_maxpool_backward(mask, y, x.shape, 3)]
    for k, call in enumerate(calls):
        got = call()
        with _General():
            want = call()
        torch.cuda.synchronize()
        assert _equal(got, want), k


@pytest.mark.gpu
def test_other_calls_are_the_general_ones_still():
    x = torch.randn(2, 3, 16, 16, device="cuda:0")
    p = pkg.division_compress(x, 8, 2, 5)
    for B in (np.int64(8), torch.tensor(8)):
        assert torch.equal(pkg.division_compress(x, B, 2, 5), p)
    par = torch.nn.Parameter(x)
    assert torch.equal(pkg.division_compress(par, 8, 2, 5), p)
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(s):
        a = pkg.division_compress(x, 8, 2, 5)
    b = pkg.division_compress(x, 8, 2, 5, stream=s)
    torch.cuda.synchronize()
    assert torch.equal(a, p) and torch.equal(b, p)
    for call, err in ((lambda: pkg.division_compress(x[:, :, ::2], 8, 2, 1), ValueError), (lambda: pkg.division_compress(x.double(), 8, 2, 1), TypeError),
                      (lambda: pkg.division_compress(x, 0, 2, 1), pkg.DivisionError), (lambda: pkg.division_compress(x, 8, 3, 1), pkg.DivisionError),
                      (lambda: pkg.division_decompress(p[:10], x.shape, 8, 2), pkg.DivisionError), (lambda: pkg.division_compress_maps([x], 8, 2, [1, 2]), ValueError),
                      (lambda: pkg.division_decompress_maps([p[:10]], [x.shape], 8, 2), pkg.DivisionError), (lambda: pkg.division_maxpool_backward(p, x, x.shape, 2), ValueError),
                      (lambda: pkg.division_compress(x, 8.0, 2, 1), Exception), (lambda: pkg.division_compress_maps([x, x[0]], 8, 2, [1, 2]), ValueError)):
        with pytest.raises(err) as native:
            call()
        with _General(), pytest.raises(err) as general:
            call()
        assert type(native.value) is type(general.value) and str(native.value) == str(general.value)


@pytest.mark.gpu
def test_other_threads_run_while_a_call_allocates():
    """The outputs of a call may have to come from the device: other Python threads do not wait for that longer than with the general calls."""
    import threading
    import time
    x = torch.zeros((64, 64, 512, 512), dtype=torch.bfloat16, device="cuda:0")
    pkg.division_relu_forward(x[:1, :1])
    torch.cuda.synchronize()
    worst, done = [0.0], []

    def count():
        last = time.perf_counter()
        while not done:
            now = time.perf_counter()
            worst[0], last = max(worst[0], now - last), now

    def waits():
        found = []
        for _ in range(8):
            torch.cuda.empty_cache()
            time.sleep(0.01)
            worst[0] = 0.0
            out = pkg.division_relu_forward(x)
            time.sleep(0.002)                                  # the other thread sees how long it waited
            found.append(worst[0])
            del out
        return found

    thread = threading.Thread(target=count)
    thread.start()
    try:
        native = waits()
        with _General():
            general = waits()
    finally:
        done.append(True)
        thread.join()
    torch.cuda.synchronize()
    assert min(native) < 5 * min(general) + 5e-5, (native, general)


# every call's work is on the stream that is current for it: recorded into a graph with the others, replayed over other inputs
@pytest.mark.gpu
@pytest.mark.parametrize("native", [True, False])
def test_calls_run_on_the_current_stream(native):
    import contextlib
    gen = torch.Generator().manual_seed(11)
    inputs = [torch.randn((3, 5, 14, 14), generator=gen).to("cuda:0") for _ in range(4)]
    x = inputs[0].clone()

    def calls():
        y, mask = pkg.division_maxpool_forward(x, 3)
        p = pkg.division_compress(x, 8, 2, 5)
        ps = pkg.division_compress_maps([x, x[:2]], 8, [2, 4], [6, 7])
        r = pkg.division_relu_forward(x)
        return [y, mask, p, *ps, *r, *pkg.division_relu_compress(x, 8, 2, 3), *pkg.division_dropout_forward(x, 0.25, 9), pkg.division_decompress(p, x.shape, 8, 2),
                *pkg.division_decompress_maps(ps, [x.shape, x[:2].shape], 8, [2, 4]), pkg.division_mask_backward(r[1], x), pkg.division_maxpool_backward(mask, y, x.shape, 3)]

    with contextlib.nullcontext() if native else _General():
        wanted = []
        for v in inputs:
            x.copy_(v)
            wanted.append([t.clone() for t in calls()])
        torch.cuda.synchronize()
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph):
            outputs = calls()
        for v, want in zip(inputs[::-1] + inputs, wanted[::-1] + wanted):
            x.copy_(v)
            graph.replay()
            torch.cuda.synchronize()
            for k, (got, ref) in enumerate(zip(outputs, want)):
                assert torch.equal(got, ref), k
            calls()
