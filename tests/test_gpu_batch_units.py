"""Dealing a batch's units to the XCDs: every unit exactly once, at unit counts
on both sides of each chunk size and at grids smaller than, equal to and larger
than one workgroup per unit.  Every pair's outputs are bitwise its single-pair
launch's (which the parity tests hold against the oracle)."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, synth
from paper_2501_10653_amd.batch import Batch, batch_cfg
from tests.gpu_util import assert_parity, oracle_for, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


# 32 x 32 images with one tile: one unit per pair
@pytest.mark.parametrize("waves", [4, 12, 36, 400, 8192, 262144])
@pytest.mark.parametrize("count", [1, 7, 9, 63, 64, 129, 1023, 2049, 4095, 4097])
def test_every_unit_once(count, waves):
    rng = np.random.default_rng(count)
    images = [synth.random_pair(32, rng, neg_frac=0.3, scale=1.0) for _ in range(5)]
    dev = [(to_dev(x), to_dev(y)) for x, y in images]
    b = Batch([(*dev[i % 5], 32) for i in range(count)], sums=True, waves=waves, inline=False)
    assert b.units == count
    b.out.fill_(-1.0)
    b.run()
    torch.cuda.synchronize()
    ref = [iqa_tiles(x, y, 32, sums=True, cfg=batch_cfg(32, 32)) for x, y in dev]
    torch.cuda.synchronize()
    assert_parity(ref[0], oracle_for(*images[0], 32), what="single launch")
    got = torch.stack([torch.cat((r.lisi.flatten(), r.auglisi.flatten(), r.sums.flatten()))
                       for r in b.results])
    want = torch.stack([torch.cat((r.lisi.flatten(), r.auglisi.flatten(), r.sums.flatten()))
                        for r in ref])[torch.arange(count) % 5]
    assert torch.equal(got.view(torch.int32), want.view(torch.int32))
