"""Python-side arguments, without a GPU: what the binding accepts for a device."""

from __future__ import annotations

import pytest
import torch

from paper_2501_10653_amd import iqa


@pytest.mark.parametrize("device", ["cuda:0", "cuda", 0, torch.device("cuda"), torch.device("cuda", 0)])
def test_devices_by_name_and_number(device, monkeypatch):
    """A device may be whatever torch.cuda.device takes: also a name or an index."""
    seen = []

    class Stream:
        cuda_stream = 4096

    class Device:
        def __init__(self, d):
            seen.append(d)

        def __enter__(self):
            seen.append("in")

        def __exit__(self, *exc):
            seen.append("out")

    monkeypatch.setattr(torch.cuda, "Stream", Stream)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda d=None: Stream())
    monkeypatch.setattr(torch.cuda, "device", Device)
    monkeypatch.setattr(iqa, "_cuda_getCurrentRawStream", lambda index: 4096 + 0 * (index << 1))
    monkeypatch.setattr(iqa, "_cuda_getDevice", lambda: 1)
    assert iqa._stream_handle(device, None) == 4096
    assert iqa._on_device(device, lambda v: v + 1, 1) == 2
    assert seen == [device, "in", "out"]
