"""fq_quantize, fq_quantize_sr and fq_gemm through the native module against the same calls through ctypes: the forms of
their arguments, their errors, the current stream; and on the CPU, what the native module leaves to the Python code."""
import ctypes as C
import os
import threading
import time
import types

import numpy as np
import pytest
import torch
from torch.overrides import TorchFunctionMode
from torch.utils._python_dispatch import TorchDispatchMode

import paper_2503_08040_amd as fq
from paper_2503_08040_amd import build

_fqnative = pytest.importorskip("paper_2503_08040_amd._fqnative", reason="the native module has not been built")

gpu = pytest.mark.gpu


def test_anything_unusual_is_left_to_the_python_code():
    x = torch.zeros((4, 8), dtype=torch.bfloat16)                 # not on the GPU
    for theta in (1.0, 1, "1", None, torch.tensor(1.0)):
        assert _fqnative.quantize(x, 1, theta, 0, 128) is None
    for first in (None, 3, torch.nn.Parameter(x), x.float(), np.zeros((4, 8)), x[0]):
        assert _fqnative.quantize(first, 1, 1.0, 0, 128) is None
        assert _fqnative.quantize_sr(first, 1, 0) is None
    a, b = fq.fq_qtensor(rows=3, cols=4), fq.fq_qtensor(rows=5, cols=4)
    args = [C.addressof(a), C.addressof(b), x]
    assert _fqnative.gemm(7, *args, None, None) is None                           # no such product
    assert _fqnative.gemm(True, *args, None, None) is None
    assert _fqnative.gemm(0, *args, None, torch.float16) is None                  # no such output
    assert _fqnative.gemm(0, *args, None, "f32") is None
    assert _fqnative.gemm(0, *args, torch.zeros(3, 5), None) is None              # not on the GPU
    with pytest.raises(TypeError):
        _fqnative.setup(1, 2)


def test_the_module_belongs_to_the_library():
    tag = build.header_flag().split('"')[1]
    assert len(tag) == 16 and _fqnative.header_tag == tag == fq.fq_header_tag()


@pytest.mark.parametrize("torch_version,header_tag,taken", [(torch.__version__, None, True), (torch.__version__, "", False),
                                                            (torch.__version__, "0123456789abcdef", False),
                                                            ("0.1", None, False)])
def test_a_module_built_for_something_else_is_not_used(torch_version, header_tag, taken, monkeypatch):
    calls = []
    other = types.SimpleNamespace(torch_version=torch_version, setup=lambda *a: calls.append(a),
                                  header_tag=_fqnative.header_tag if header_tag is None else header_tag)
    monkeypatch.setattr(fq, "_fqnative", other)
    monkeypatch.setattr(fq, "_native", None)
    fq._native_setup()
    assert (fq._native is other) == taken == (len(calls) == 1)


def test_the_module_is_rebuilt_with_the_header(tmp_path, monkeypatch):
    sources = {"SOURCES": "a.hip", "HEADERS": "a.h", "HEADER": "fq.h", "NATIVE_SOURCE": "m.cpp", "LIB": "l.so", "NATIVE": "m.so"}
    for name, f in sources.items():
        path = tmp_path / f
        path.write_text("")
        os.utime(path, (100, 200 if f.endswith(".so") else 100))
        monkeypatch.setattr(build, name, [str(path)] if name in ("SOURCES", "HEADERS") else str(path))
    built = []
    monkeypatch.setattr(build, "_build_library", lambda flags: built.append("library"))
    monkeypatch.setattr(build, "build_native", lambda: built.append("module"))
    assert not build.stale() and build.build(force=False) and built == []
    os.utime(tmp_path / "m.cpp", (300, 300))
    assert build.stale() and build.build(force=False) and built == ["module"]
    os.utime(tmp_path / "m.so", (400, 400))
    assert not build.stale()
    for h in ("fq.h", "a.h"):                       # the library's headers are listed, fq.h among them
        os.utime(tmp_path / h, (500, 500))
    assert build.stale() and build.build(force=False) and built == ["module", "library", "module"]
    assert build.build() and built[3:] == ["library", "module"]


@pytest.fixture
def structs():
    """Addresses of two structs of 3 and 5 rows."""
    keep = [fq.fq_qtensor(rows=n, cols=4) for n in (3, 5)]
    yield [C.addressof(s) for s in keep]


class _Raises(TorchDispatchMode):
    """Every operation raises the given exception."""

    def __init__(self, error):
        super().__init__()
        self.error = error

    def __torch_dispatch__(self, func, types, args=(), kwargs=None):
        raise self.error


@pytest.mark.parametrize("error", [torch.OutOfMemoryError("no memory left"), KeyError("key"), RuntimeError("text"),
                                   KeyboardInterrupt(), FloatingPointError("a", 2)], ids=lambda e: type(e).__name__)
def test_errors_of_the_outputs_allocation_are_torchs(error, structs):
    x = torch.zeros(1)
    caught = []
    for allocate in (lambda: torch.empty((3, 5)), lambda: _fqnative.gemm(0, *structs, x, None, None)):
        with _Raises(error), pytest.raises(BaseException) as e:
            allocate()
        caught.append((type(e.value), e.value.args))
    assert caught[0] == caught[1] == (type(error), error.args)


def test_an_allocation_that_fails_is_reported_as_torch_reports_it(structs):
    huge = [fq.fq_qtensor(rows=2 ** 31 - 1, cols=1) for _ in range(2)]
    caught = []
    for allocate in (lambda: torch.empty((2 ** 31 - 1, 2 ** 31 - 1)),
                     lambda: _fqnative.gemm(0, *(C.addressof(h) for h in huge), torch.zeros(1), None, None)):
        with pytest.raises(RuntimeError) as e:
            allocate()
        caught.append((type(e.value), str(e.value)))
    assert caught[0] == caught[1]


@pytest.fixture
def no_launch():
    """The native module as if the current device could not be had: a call raises LookupError in front of its launch."""
    def device():
        raise LookupError
    _fqnative.setup(0, 0, 0, device, device)
    yield
    fq._native_setup()


class _Sees(TorchFunctionMode):
    """Notes the functions of torch that are called."""

    def __init__(self):
        super().__init__()
        self.seen = []

    def __torch_function__(self, func, types, args=(), kwargs=None):
        self.seen.append(func)
        return func(*args, **(kwargs or {}))


def test_a_mode_that_sees_torchs_functions_sees_the_allocation(structs, no_launch):
    x = torch.zeros(1)
    with _Sees():
        assert _fqnative.gemm(0, *structs, x, None, None) is None


def test_other_threads_run_while_the_output_is_allocated(no_launch):
    """As with torch.empty; the allocation takes long here because torch's deterministic mode fills it."""
    n = 16000
    q, over, ticks = fq.fq_qtensor(rows=n, cols=1), threading.Event(), []

    def tick():
        while not over.wait(0.001):
            ticks.append(time.perf_counter())
    during = []
    thread = threading.Thread(target=tick)
    thread.start()
    torch.use_deterministic_algorithms(True)
    try:
        for allocate in (lambda: torch.empty((n, n)),
                         lambda: _fqnative.gemm(0, C.addressof(q), C.addressof(q), torch.zeros(1), None, None)):
            start = time.perf_counter()
            try:
                allocate()
            except LookupError:
                pass
            end = time.perf_counter()
            during.append(sum(start < t < end for t in ticks))
    finally:
        torch.use_deterministic_algorithms(False)
        over.set()
        thread.join()
    assert min(during) >= 5, during


@pytest.fixture
def both(monkeypatch):
    """Runs a call through the native module (and makes sure of it) and through ctypes."""
    fq.QTensor(1, 1)
    assert fq._native is _fqnative

    def run(call):
        out = []
        for native in (True, False):
            with monkeypatch.context() as m:
                if not native:
                    m.setattr(fq, "_native", None)
                try:
                    out.append(call())
                except Exception as e:                     # compared, not hidden
                    out.append((type(e), getattr(e, "status", None)))
        return out
    return run


def _state(q):
    names = ["codes", "scales", "mask"] + (["codes_t"] if q.want_transposed else [])
    return [q.view(n).clone() for n in names]


@gpu
@pytest.mark.parametrize("shape,pitch", [((1, 8), 8), ((1, 300), 512), ((130, 260), 264), ((7, 1), 1), ((0, 5), 5)])
def test_quantize_forms(shape, pitch, both):
    g = torch.Generator(device="cuda").manual_seed(3)
    x = torch.randn((shape[0], pitch), device="cuda", generator=g).bfloat16()[:, :shape[1]]
    q = fq.QTensor(*shape, want_transposed=True)
    q.storage.zero_()

    def nearest(theta):
        fq.fq_quantize(x, fq.FQ_CRIT_ABSMAX_GT, theta, out=q)
        return _state(q)

    def stochastic(seed):
        fq.fq_quantize_sr(x, seed, out=q)
        return _state(q)
    for f, values in ((nearest, (0.5, 1, float("inf"))), (stochastic, (5, -1, 2 ** 64 + 9))):
        for v in values:
            n, p = both(lambda: f(v))
            assert len(n) == len(p) and all(torch.equal(s, t) for s, t in zip(n, p))


@gpu
@pytest.mark.parametrize("op", [fq.FQ_OP_NT, fq.FQ_OP_NN, fq.FQ_OP_TN])
def test_gemm_forms(op, both):
    g = torch.Generator(device="cuda").manual_seed(4)
    sa, sb = {0: ((33, 200), (70, 200)), 1: ((33, 200), (200, 70)), 2: ((200, 33), (200, 70))}[op]
    a, b = (fq.fq_quantize(torch.randn(s, device="cuda", generator=g).bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0,
                           want_transposed=True) for s in (sa, sb))
    wide = torch.zeros((33, 96), device="cuda")
    for kw in ({}, {"out_dtype": torch.float32}, {"out_dtype": torch.bfloat16}, {"out": wide[:, 8:78]},
               {"out": torch.zeros((33, 70), device="cuda", dtype=torch.bfloat16)}):
        n, p = both(lambda: fq.fq_gemm(op, a, b, **kw).clone())
        assert n.dtype == p.dtype and n.device == p.device and n.shape == p.shape and torch.equal(n, p)
    assert fq.fq_gemm(op, a, b, out=wide[:, 8:78]).data_ptr() == wide[:, 8:78].data_ptr()
    for kw in ({"out_dtype": torch.float16}, {"out": torch.zeros((33, 71), device="cuda")},
               {"out": torch.zeros((70, 33), device="cuda").t()}):
        n, p = both(lambda: fq.fq_gemm(op, a, b, **kw))
        assert n == p and isinstance(n, tuple)


@gpu
def test_errors_are_the_same(both):
    x = torch.randn((256, 256), device="cuda").bfloat16()
    q, none = fq.QTensor(256, 256), fq.QTensor(256, 256, capacity=0)
    for call in (lambda: fq.fq_quantize(x, fq.FQ_CRIT_ABSMAX_GT, 1.0, out=none), lambda: fq.fq_quantize(x, 9, 1.0, out=q),
                 lambda: fq.fq_quantize(x[:128], 0, 1.0, out=q), lambda: fq.fq_quantize(x.float(), 0, 1.0, out=q),
                 lambda: fq.fq_quantize(x.t(), 0, 1.0, out=q), lambda: fq.fq_quantize(x, 0, "1", out=q),
                 lambda: fq.fq_quantize_sr(x, 1.5, out=q), lambda: fq.fq_quantize_sr(x[:, :8], 1, out=q),
                 lambda: fq.fq_gemm(5, q, q), lambda: fq.fq_gemm(fq.FQ_OP_TN, q, q)):
        n, p = both(call)
        assert n == p and isinstance(n, tuple), (n, p)


@gpu
def test_the_current_stream_is_used(both):
    x = torch.randn((512, 512), device="cuda").bfloat16()
    q = fq.fq_quantize(x, fq.FQ_CRIT_NONE, 0.0, capacity=0)
    want = fq.fq_gemm(fq.FQ_OP_NT, q, q)
    torch.cuda.synchronize()
    side = torch.cuda.Stream()

    def captured():                    # a call on any other stream would not be in the graph
        graph = torch.cuda.CUDAGraph()
        out = torch.zeros_like(want)
        with torch.cuda.graph(graph, stream=side):
            fq.fq_gemm(fq.FQ_OP_NT, q, q, out=out)
        for _ in range(3):
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
        return out
    n, p = both(captured)
    assert torch.equal(n, p)


@gpu
def test_out_of_memory_keeps_its_type(both):
    """The output does not fit what torch may take of the card: the allocator refuses, nothing is asked of the driver."""
    n = 40000                                                    # 6.4 GB
    q = fq.fq_quantize(torch.zeros((n, 8), device="cuda", dtype=torch.bfloat16), fq.FQ_CRIT_NONE, 0.0, capacity=0)
    torch.cuda.empty_cache()
    torch.cuda.set_per_process_memory_fraction(0.01)
    try:
        results = both(lambda: fq.fq_gemm(fq.FQ_OP_NT, q, q))
    finally:
        torch.cuda.set_per_process_memory_fraction(1.0)
    assert results == [(torch.OutOfMemoryError, None)] * 2


@gpu
def test_a_mode_sees_the_outputs_allocation(both):
    q = fq.fq_quantize(torch.randn((32, 32), device="cuda").bfloat16(), fq.FQ_CRIT_NONE, 0.0, capacity=0)

    def empties():
        with _Sees() as mode:
            fq.fq_gemm(fq.FQ_OP_NT, q, q)
        return mode.seen.count(torch.empty)
    assert both(empties) == [1, 1]
