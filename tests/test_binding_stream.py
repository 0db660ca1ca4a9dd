"""The stream handle that the binding passes on: a given stream's own, else the
handle of torch's current one -- by torch's function for the handle alone, or
by the documented Stream object where torch does not have it."""
from types import SimpleNamespace

import torch

import paper_2301_13062_amd as cp


def test_given_stream():
    assert cp._stream_ptr(SimpleNamespace(cuda_stream=17)) == 17


def test_current_stream(monkeypatch):
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(cp, "_raw_stream", lambda device: 100 + device)
    assert cp._stream_ptr(None) == 103


def test_current_stream_without_the_handle_function(monkeypatch):
    monkeypatch.setattr(cp, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: SimpleNamespace(cuda_stream=41))
    assert cp._stream_ptr(None) == 41
