"""The Python layer without a GPU: what it hands to the C library, which is replaced by a recorder here."""
import ctypes as C
import types

import pytest
import torch

import paper_2503_08040_amd as fq


class _Recorder:
    """Stands for the loaded library: notes every call and reports success."""

    def __init__(self):
        self.calls = []

    def __getattr__(self, name):
        def call(*args):
            self.calls.append((name, args))
            return fq.FQ_OK
        return call


@pytest.fixture
def recorder(monkeypatch):
    r = _Recorder()
    monkeypatch.setattr(fq, "_lib", r)
    return r


def _scalars():
    x = types.SimpleNamespace(dtype=torch.bfloat16, is_cuda=True, shape=(1, 8), dim=lambda: 2,
                              stride=lambda: (8, 1), data_ptr=lambda: 256)
    out = types.SimpleNamespace(block=fq.FQ_BLOCK, _ref=C.byref(fq.fq_qtensor()))
    stream = types.SimpleNamespace(cuda_stream=0)
    m = torch.zeros((2, 8), dtype=torch.bfloat16)
    return {"theta": lambda v: fq.fq_quantize(x, fq.FQ_CRIT_ABSMAX_GT, v, out=out, stream=stream),
            "eps": lambda v: fq.fq_rmsnorm_forward(m, m[0].clone(), v, stream=stream)}


@pytest.mark.parametrize("name", ["theta", "eps"])
def test_a_number_is_taken_and_a_text_refused(name, recorder):
    call = _scalars()[name]
    for v in (2, 2.5, torch.tensor(0.5), True):
        call(v)
    values = [a.value if isinstance(a, C.c_float) else a for _, args in recorder.calls for a in args
              if isinstance(a, (float, C.c_float))]
    assert values == [2.0, 2.5, 0.5, 1.0]
    n = len(recorder.calls)
    for v in ("2.5", b"2.5", None, 1j):
        with pytest.raises(TypeError):
            call(v)
    assert len(recorder.calls) == n


def test_the_current_stream_without_torchs_internal_names(monkeypatch):
    """The quick way to the current stream's handle uses names torch does not document: a torch that
    lacks them is asked through torch.cuda.current_stream()."""
    public = types.SimpleNamespace(current_stream=lambda: types.SimpleNamespace(cuda_stream=77))
    quick = types.SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda dev: 100 + dev)
    for internal, want in ((types.SimpleNamespace(), 77), (quick, 103)):
        monkeypatch.setattr(fq, "_torch", types.SimpleNamespace(_C=internal, cuda=public))
        monkeypatch.setattr(fq, "_current_stream", None, raising=False)
        assert fq._stream_ptr(None) == want
    assert fq._stream_ptr(types.SimpleNamespace(cuda_stream=5)) == 5
