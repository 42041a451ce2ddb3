"""What the binding does on the host alone: no GPU, no library call."""
import types

import pytest
import torch

from paper_2607_00466_amd import binding as B


@pytest.mark.parametrize("stream", [0, 1, True, 1 << 40, "0", 0.0])
def test_only_stream_objects_are_streams(stream):
    # 0 would be the null stream and any other number a pointer the library follows
    with pytest.raises(AttributeError):
        B._stream(stream)


def test_stream_addresses(monkeypatch):
    assert B._stream(types.SimpleNamespace(cuda_stream=1 << 40)) == 1 << 40
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    monkeypatch.setattr(B, "_raw_stream", lambda device: 100 + device)
    assert B._stream(None) == 103
    # a torch without the raw lookup
    monkeypatch.setattr(B, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: types.SimpleNamespace(cuda_stream=77))
    assert B._stream(None) == 77
