"""The stream that calls go to, with and without the short way to its handle that torch does not document. CPU only for the choice
itself; on a GPU both ways name the same stream."""
import types

import pytest
import torch

from paper_2604_06694_amd import binding


@pytest.mark.parametrize("missing", ["_raw_stream", "_raw_device"])
def test_without_the_short_way(monkeypatch, missing):
    monkeypatch.setattr(binding, missing, None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert binding._stream() == 1234


def test_the_short_way_asks_for_the_current_device(monkeypatch):
    monkeypatch.setattr(binding, "_raw_stream", lambda device: 100 + device)
    monkeypatch.setattr(binding, "_raw_device", lambda: 3)
    assert binding._stream() == 103


@pytest.mark.gpu
def test_both_ways_name_the_current_stream():
    for stream in (torch.cuda.default_stream(), torch.cuda.Stream()):
        with torch.cuda.stream(stream):
            assert binding._stream() == torch.cuda.current_stream().cuda_stream == stream.cuda_stream
