"""The stream that a call without one runs on: torch's current stream, from the
raw handle where this torch has it, from the public object otherwise."""
import types

import pytest


def test_public_stream_object_where_the_raw_handle_is_missing(monkeypatch):
    import torch

    from paper_2609_32237_amd import torch_api

    monkeypatch.setattr(torch_api, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda *a: types.SimpleNamespace(cuda_stream=42))
    assert torch_api._stream(None) == 42


@pytest.mark.gpu
def test_current_stream(monkeypatch):
    import torch

    from paper_2609_32237_amd import torch_api

    side = torch.cuda.Stream()
    for raw in (torch_api._raw_stream, None):
        monkeypatch.setattr(torch_api, "_raw_stream", raw)
        assert torch_api._stream(None) == torch.cuda.current_stream().cuda_stream
        with torch.cuda.stream(side):
            assert torch_api._stream(None) == side.cuda_stream
        assert torch_api._stream(side) == side.cuda_stream
