"""Which gathers are ordered between streams: a gather runs on the lattice's
stream, and the caller's current stream waits for it unless the two are one,
handle and device alike (default streams of all devices share a handle)."""
import types

import pytest
import torch

from paper_0707_1581_amd import lb


def _stream(device_index, handle):
    return types.SimpleNamespace(device_index=device_index, cuda_stream=handle)


@pytest.mark.parametrize("index,stream,same", [
    (0, (0, 0), True),
    (1, (0, 0), False),   # made on device 0, gathered with device 1 current: both default streams
    (0, (1, 0), False),
    (0, (0, 7), False),
    (1, (1, 0), True),
])
def test_current_stream_by_device_and_handle(monkeypatch, index, stream, same):
    monkeypatch.setattr(lb, "_raw_stream", lambda i: 0)
    assert lb._is_current(_stream(*stream), index) is same


def test_without_raw_handles(monkeypatch):
    here = _stream(0, 0)
    monkeypatch.setattr(lb, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda index: here)
    assert lb._is_current(here, 0)
    assert not lb._is_current(_stream(0, 1), 0)
