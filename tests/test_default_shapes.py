"""The built-in launch shapes over many sizes and alignments (CPU): always a
configuration that the library accepts, never more parts than the fixed
scratch array and a workgroup's LDS hold."""

from __future__ import annotations

import ctypes
import random

from paper_2501_10653_amd import _lib
from paper_2501_10653_amd._lib import IqaPair, LaunchCfg


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


def test_eight_waves_for_a_workgroup_on_most_cus():
    lib = _lib.load()
    c = LaunchCfg()
    for ns, NT, eight in [(10, 160, False), (11, 160, True), (11, 200, False), (12, 160, True), (16, 160, True), (17, 160, False),
                          (12, 120, False), (15, 128, True), (12, 320, True), (12, 400, False),
                          (12, 164, False)]:
        assert lib.iqa_default_cfg(ns * NT, NT, 256, 256, ctypes.byref(c)) == 0
        assert (c.waves == 8 and c.ksplit == 1) == eight, (ns, NT, c.as_dict())
    for ns, NT, sixteen in [(1, 128, True), (14, 128, True), (15, 128, False), (2, 120, False),
                            (8, 112, True), (8, 96, False), (3, 160, False)]:
        assert lib.iqa_default_cfg(ns * NT, NT, 256, 256, ctypes.byref(c)) == 0
        assert (c.waves == 16 and c.ksplit == 1) == sixteen, (ns, NT, c.as_dict())


def test_odd_batches_take_what_a_single_launch_of_any_address_quads_takes():
    """iqa_odd_batch_describe accepts exactly the pairs whose default shape is
    unsplit quads at any address, with one unit per workgroup of that launch."""
    lib = _lib.load()
    rng = random.Random(12)
    c, units = LaunchCfg(), ctypes.c_int64()
    desc = ctypes.create_string_buffer(_lib.BATCH_DESC_BYTES)
    taken = 0
    for _ in range(4000):
        NT = int(2 ** rng.uniform(0, 9))
        N = NT * max(1, int(2 ** rng.uniform(0, 7)))
        x, y = (256 + 4 * rng.choice((0, 0, 1, 2, 3)) for _ in range(2))
        pair = IqaPair(x, y, N, NT, 5e-7, 1e-6, 1e-6, 1e-6, 4096, 8192, None)
        st = lib.iqa_odd_batch_describe(ctypes.byref(pair), 1, desc, ctypes.byref(units))
        assert lib.iqa_default_cfg(N, NT, x, y, ctypes.byref(c)) == 0
        if c.vec < 4 and NT >= 4 and c.ksplit == 1:
            taken += 1
            assert st == 0
            assert units.value == lib.iqa_launch_workgroups(N, NT, ctypes.byref(c))
        else:
            assert _lib.STATUS_NAMES[st] == "IQA_ERR_CONFIG"
    assert 1000 < taken < 3500
    pair.x = 257
    st = lib.iqa_odd_batch_describe(ctypes.byref(pair), 1, desc, ctypes.byref(units))
    assert _lib.STATUS_NAMES[st] == "IQA_ERR_ALIGN"
    assert lib.iqa_odd_tiles_batched(None, 1, 1, None) == 1
    assert lib.iqa_odd_tiles_batched(4096, 0, 1, None) == 2
    assert lib.iqa_odd_tiles_batched(4096, 1, 0, None) == 2
    assert lib.iqa_odd_tiles_batched(4104, 1, 1, None) == 3
