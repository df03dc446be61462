"""The built-in launch shapes over many sizes and alignments (CPU): always a
configuration that the library accepts, never more parts than the fixed
scratch array and a workgroup's LDS hold."""

from __future__ import annotations

import ctypes
import random

from paper_2501_10653_amd import _lib
from paper_2501_10653_amd._lib import LaunchCfg


def test_default_shapes_are_accepted_and_bounded():
    lib = _lib.load()
    rng = random.Random(11)
    c = LaunchCfg()
    split = 0
    for _ in range(20000):
        NT = int(2 ** rng.uniform(0, 14))
        N = NT * (1 if rng.random() < 0.2 else max(1, int(2 ** rng.uniform(0, 9))))
        if N > 1 << 17:
            continue
        x, y = (256 + 4 * rng.choice((0, 0, 0, 1, 2)) for _ in range(2))
        assert lib.iqa_default_cfg(N, NT, x, y, ctypes.byref(c)) == 0
        assert lib.iqa_check_cfg(N, NT, ctypes.byref(c)) == 0, (N, NT, c.as_dict())
        if c.ksplit > 1:
            split += 1
            parts = (N // NT) ** 2 * c.ksplit
            assert parts * 128 <= _lib.NOALLOC_SCRATCH_BYTES - (64 << 10) or parts > 1024
            assert parts * 16 <= _lib.NOALLOC_SCRATCH_BYTES - (64 << 10), (N, NT, c.as_dict())
            assert c.ksplit * c.waves * 16 <= 64 << 10
            assert c.seg * c.rp == 64 and c.waves in (1, 2, 4, 8, 16)
    assert split > 100
