"""The Python binding's own conversions, checked without a GPU.

For the calls themselves the library is replaced by a recorder and the tensors
are host tensors that say they are on the device: what is looked at is what the
binding hands over or refuses, nothing is launched.
"""

import ctypes
import types

import pytest
import torch

import paper_2607_16190_amd as fva


class DeviceTensor(torch.Tensor):
    is_cuda = True


class Recorder:
    """Stands for the loaded library: host queries go through, calls are recorded."""

    def __init__(self, lib):
        self._lib = lib
        self.calls = []

    def __getattr__(self, name):
        if name.endswith("_size") or name.endswith("_words"):
            return getattr(self._lib, name)

        def call(*args):
            self.calls.append((name, args))
            return fva.FVA_OK

        return call


@pytest.fixture
def recorder(monkeypatch):
    r = Recorder(fva.lib)
    monkeypatch.setattr(fva, "lib", r)
    return r


STREAM = types.SimpleNamespace(cuda_stream=0x77)


def test_current_stream_without_the_raw_accessor(monkeypatch):
    # the accessor is a private function of torch: without it the public object's pointer is used
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0x1234))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert fva._stream_ptr(None) == 0x1234


def test_given_stream_is_used(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1 / 0, raising=False)
    assert fva._stream_ptr(STREAM) == 0x77


def attention_calls():
    """The three attention calls on a two-block clip, as functions of the scale."""

    def tensor(*shape, dtype):
        return torch.zeros(shape, dtype=dtype).as_subclass(DeviceTensor)

    t = fva.Tiling(1, 8, 16, 1, 8, 8)
    q, k, v, out = (tensor(1, 1, 128, 128, dtype=torch.bfloat16) for _ in range(4))
    mask = tensor(1, 1, 2, 2, dtype=torch.uint8)
    counts, kv = tensor(1, 1, 2, dtype=torch.int32), tensor(1, 1, 2, 2, dtype=torch.int32)
    v8, vexp = tensor(1, 1, 2, 128, 128, dtype=torch.uint8), tensor(1, 1, 128, dtype=torch.int32)
    return {
        "fva_attn": lambda s: fva.fva_attn(q, k, v, t, mask, counts, kv, scale=s, out=out, stream=STREAM),
        "fva_attn_noalloc": lambda s: fva.fva_attn_noalloc(q, k, v, t, counts, kv, out, scale=s, stream=STREAM),
        "fva_attn_fp8v": lambda s: fva.fva_attn_fp8v(q, k, v8, vexp, t, mask, counts, kv, scale=s, out=out,
                                                     stream=STREAM),
    }


@pytest.mark.parametrize("name", ["fva_attn", "fva_attn_noalloc", "fva_attn_fp8v"])
def test_scale_is_a_number(recorder, name):
    call = attention_calls()[name]
    call(0.125)
    (done,) = recorder.calls
    assert done[0] == name and [a.value for a in done[1] if isinstance(a, ctypes.c_float)] == [0.125]
    for text in ("0.125", "nan", "inf"):
        with pytest.raises(TypeError):
            call(text)
    assert len(recorder.calls) == 1
