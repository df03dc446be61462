"""Python-side arguments, without a GPU: what the binding accepts for a device."""

from __future__ import annotations

import os
import subprocess
import sys

import pytest
import torch

from paper_2501_10653_amd import iqa

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


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


def test_the_package_imports_on_a_torch_without_gpu_support():
    """A CPU build of torch lacks the private names of the short host path: the
    package, synth and the plain helpers import there all the same, and a call
    fails with torch's own words."""
    code = (
        "import torch\n"
        "for n in [n for n in dir(torch._C) if n.startswith('_cuda_')]:\n"
        "    delattr(torch._C, n)\n"
        "import paper_2501_10653_amd as p\n"
        "from paper_2501_10653_amd import batch, serve, synth\n"
        "assert p.default_D(1e-6) > 0\n"
        "try:\n"
        "    p.merge_tiles(torch.zeros(4, 4), 2)\n"
        "except Exception as e:\n"
        "    assert not isinstance(e, (NameError, TypeError)), repr(e)\n"
        "else:\n"
        "    raise AssertionError('ran without a GPU')\n")
    subprocess.run([sys.executable, "-c", code], check=True, cwd=ROOT)


@pytest.mark.parametrize("stream", [None, 0])
def test_sums_in_host_memory_are_refused_as_such(stream):
    """Also where there is no GPU: the words are about the tensor."""
    with pytest.raises(ValueError, match="Expected a cuda device, but got: cpu"):
        iqa.merge_tiles(torch.zeros(4, 4), 2, stream=stream)
