"""Lanes per tile of the built-in rule for quads at any address in rows of 13 to 16
quads (CPU): sixteen where they make 256 workgroups, or more than 384 and at most
512."""

from __future__ import annotations

import ctypes

import pytest

from paper_2501_10653_amd import _lib
from paper_2501_10653_amd._lib import LaunchCfg


@pytest.mark.parametrize("N,NT,off,lanes", [
    (1600, 50, 0, 16), (1800, 50, 0, 32), (2000, 50, 0, 16), (2200, 50, 0, 16), (2350, 50, 0, 32), (4000, 50, 0, 32),
    (1960, 49, 0, 16), (2303, 49, 0, 32), (2332, 53, 0, 16), (2385, 53, 0, 32), (1961, 53, 0, 32),
    (2394, 57, 0, 16), (3990, 57, 0, 32), (2646, 63, 0, 16), (2835, 63, 0, 32),
    (2560, 64, 4, 16), (2880, 64, 4, 32), (1980, 45, 0, 32), (1804, 41, 0, 32)])
def test_sixteen_lanes(N, NT, off, lanes):
    c = LaunchCfg()
    assert _lib.load().iqa_default_cfg(N, NT, 256 + off, 256 + off, ctypes.byref(c)) == 0
    assert c.seg * c.rp == lanes and c.ksplit == 1
