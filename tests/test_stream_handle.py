"""The current stream's handle without the two functions of torch that are not
part of its interface."""
from types import SimpleNamespace

import pytest

from paper_1308_1419_amd import tdmap


@pytest.mark.parametrize("functions", [{}, {"_cuda_getDevice": lambda: 0},
                                       {"_cuda_getCurrentRawStream": lambda device: 5}])
def test_stream_without_the_raw_handle(monkeypatch, functions):
    cuda = SimpleNamespace(is_initialized=lambda: True,
                           current_stream=lambda: SimpleNamespace(cuda_stream=41))
    monkeypatch.setattr(tdmap, "_torch_module", SimpleNamespace(cuda=cuda, _C=SimpleNamespace(**functions)))
    assert tdmap._stream() == 41


def test_stream_by_the_raw_handle(monkeypatch):
    cuda = SimpleNamespace(is_initialized=lambda: True)
    raw = SimpleNamespace(_cuda_getDevice=lambda: 3, _cuda_getCurrentRawStream=lambda device: 100 + device)
    monkeypatch.setattr(tdmap, "_torch_module", SimpleNamespace(cuda=cuda, _C=raw))
    assert tdmap._stream() == 103
