"""The stream handle that the binding passes is torch's current stream's, of the
current device or a given one, also where torch lacks the calls that return
it directly."""
import types

import pytest
import torch

from paper_2106_11143_amd import api


@pytest.mark.parametrize("gone", ["_raw_stream", "_raw_device"])
def test_without_the_direct_calls(monkeypatch, gone):
    asked = []

    def current_stream(device=None):
        asked.append(device)
        return types.SimpleNamespace(cuda_stream=1234)

    monkeypatch.setattr(torch.cuda, "current_stream", current_stream)
    monkeypatch.setattr(api, gone, None)
    assert api._stream() == 1234
    assert api._stream(torch.device("cuda:0")) == 1234
    assert asked == [None, torch.device("cuda:0")]


def test_direct_calls(monkeypatch):
    monkeypatch.setattr(api, "_raw_device", lambda: 3)
    monkeypatch.setattr(api, "_raw_stream", lambda index: 100 + index)
    assert [api._stream(), api._stream(torch.device("cuda:1")), api._stream(torch.device("cuda"))] == [103, 101, 103]


@pytest.mark.gpu
def test_is_the_current_stream():
    side = torch.cuda.Stream()
    for dev in (None, torch.device("cuda"), torch.device("cuda:0")):
        assert api._stream(dev) == torch.cuda.current_stream(dev).cuda_stream
        with torch.cuda.stream(side):
            assert api._stream(dev) == side.cuda_stream
