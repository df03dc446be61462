"""Batches of pairs the quads of the batch kernel do not fit (N_T not a multiple
of 4, images off a 16-byte boundary): one launch for all that iqa_tiles would not
split, bitwise its results, eager and captured; the rest still launched alone."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, synth
from paper_2501_10653_amd.batch import Batch
from tests.gpu_util import assert_parity, oracle_for, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]

# (N, N_T, floats off a 16-byte boundary)
ODD = [(5, 5, 0), (90, 6, 0), (77, 7, 1), (81, 9, 0), (500, 10, 0), (1000, 25, 3), (256, 32, 1),
       (512, 64, 2), (225, 45, 0), (700, 50, 0), (1030, 103, 0)]
WIDE = (4112, 257, 0)   # rows of more quads than a wave has lanes
ALONE = [(375, 375, 0), (260, 130, 0), (640, 160, 3), (12, 2, 0), (9, 3, 0), (7, 1, 0)]


def _pair(N, off, rng):
    x, y = synth.random_pair(N, rng, neg_frac=0.3, nan_frac=0.01, scale=1.0)
    dev = torch.zeros(2, N * N + 4, device="cuda")
    views = [dev[k, off:off + N * N].view(N, N) for k in range(2)]
    if off == 0:
        views = [to_dev(x), to_dev(y)]
    else:
        views[0].copy_(to_dev(x))
        views[1] = to_dev(y)
    return (x, y), views


@pytest.mark.parametrize("shapes,quads", [(ODD, 1), (ODD + ALONE, 0), (ODD[:1], 0), (ODD[1:3] + [WIDE], 2),
                                          (ODD * 9, 0)])
def test_odd_pairs_share_a_launch(shapes, quads):
    rng = np.random.default_rng(len(shapes))
    host, dev = [], []
    for N, NT, off in shapes + [(128, 32, 0)] * quads:
        h, d = _pair(N, off, rng)
        host.append((*h, NT))
        dev.append((*d, NT))
    b = Batch(dev, sums=True, waves=4)
    odd = sum(s not in ALONE for s in shapes)
    assert b.odd_count == (odd if odd > 1 else 0)
    assert len(b.alone) == len(shapes) - b.odd_count
    want = [iqa_tiles(x, y, NT, sums=True) for x, y, NT in dev[:len(shapes)]]
    graph = b.capture() if not any(s in ALONE for s in shapes) else None
    for replay in range(4):
        b.out.fill_(-1.0)
        torch.cuda.synchronize()
        b.run() if replay == 0 or graph is None else graph.replay()
        torch.cuda.synchronize()
        for i, w in enumerate(want):
            for k in ("lisi", "auglisi", "sums"):
                got = getattr(b.results[i], k)
                assert torch.equal(got.view(torch.int32), getattr(w, k).view(torch.int32)), (i, k)
    for (x, y, NT), res in zip(host[:len(ODD) + 6], b.results):
        assert_parity(res, oracle_for(x, y, NT), what=f"{x.shape[0]}/{NT}")
