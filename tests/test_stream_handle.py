"""Host: the handle of the current stream that the binding passes on, by torch's
raw getter where there is one and through a Stream object where there is not."""
import types

import pytest
import torch

from paper_2603_05493_amd import wb


def test_without_the_raw_getter(monkeypatch):
    monkeypatch.setattr(wb, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=1234))
    assert wb._stream() == 1234


def test_with_the_raw_getter(monkeypatch):
    monkeypatch.setattr(wb, "_raw_stream", lambda device: 100 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert wb._stream() == 103


@pytest.mark.gpu
def test_follows_the_current_stream():
    side = torch.cuda.Stream()
    outer = wb._stream()
    assert outer == torch.cuda.current_stream().cuda_stream
    with torch.cuda.stream(side):
        assert wb._stream() == side.cuda_stream != outer
    assert wb._stream() == outer
