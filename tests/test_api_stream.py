"""The stream that the Python entry points enqueue on is torch's current one,
also where torch lacks the functions that name it cheaply."""
import types

import pytest
import torch

from paper_2408_05235_amd import api


@pytest.mark.parametrize("gone", ["_raw_stream", "_raw_device"])
def test_without_the_raw_functions(monkeypatch, gone):
    monkeypatch.setattr(api, gone, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert api._stream() == 1234


@pytest.mark.gpu
def test_both_name_the_current_stream(gpu, monkeypatch):
    side = torch.cuda.Stream()
    for stream in (torch.cuda.current_stream(), side):
        with torch.cuda.stream(stream):
            assert api._stream() == stream.cuda_stream
            with monkeypatch.context() as m:
                m.setattr(api, "_raw_stream", None)
                assert api._stream() == stream.cuda_stream
