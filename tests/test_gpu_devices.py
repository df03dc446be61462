"""A batch and iqa_prepare on a device given by name or index."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, prepare, synth
from paper_2501_10653_amd.batch import Batch, batch_cfg
from tests.gpu_util import requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("device", ["cuda:0", "cuda", 0, torch.device("cuda")])
def test_device_by_name_or_index(device):
    x, y = (to_dev(a) for a in synth.random_pair(256, np.random.default_rng(2), scale=1.0))
    xo, yo = (t[:250, :250].contiguous() for t in (x, y))
    b = Batch([(x, y, 32), (xo, yo, 25)], device=device)
    b.run()
    prepare(1024, 256, device=device)
    want = [iqa_tiles(x, y, 32, cfg=batch_cfg(256, 32)), iqa_tiles(xo, yo, 25)]
    torch.cuda.synchronize()
    for r, w in zip(b.results, want):
        assert torch.equal(r.lisi, w.lisi) and torch.equal(r.auglisi, w.auglisi)
