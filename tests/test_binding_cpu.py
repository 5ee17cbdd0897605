"""The Python binding's own conversions, checked without a GPU."""

import types

import torch

import paper_2607_16190_amd as fva


def test_current_stream_without_the_raw_accessor(monkeypatch):
    # the accessor is a private function of torch: without it the public object's pointer is used
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 0)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=0x1234))
    monkeypatch.delattr(torch._C, "_cuda_getCurrentRawStream", raising=False)
    assert fva._stream_ptr(None) == 0x1234


def test_given_stream_is_used(monkeypatch):
    monkeypatch.setattr(torch._C, "_cuda_getCurrentRawStream", lambda d: 1 / 0, raising=False)
    assert fva._stream_ptr(types.SimpleNamespace(cuda_stream=0x77)) == 0x77
