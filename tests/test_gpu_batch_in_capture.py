"""A batch made and run while torch captures a graph: up to 16 quads pairs and any
odd ones need no copy to the device, which a capture does not allow."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import synth
from paper_2501_10653_amd.batch import Batch
from tests.gpu_util import requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("shapes", [[(256, 32), (250, 25), (225, 45)], [(90, 6), (77, 7), (81, 9)],
                                    [(128, 32), (512, 64)]])
def test_made_under_capture(shapes):
    rng = np.random.default_rng(len(shapes) + shapes[0][0])
    pairs = [(*(to_dev(a) for a in synth.random_pair(N, rng, neg_frac=0.3, scale=1.0)), NT)
             for N, NT in shapes]
    want = Batch(pairs, sums=True)
    want.run()
    torch.cuda.synchronize()
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g):
        b = Batch(pairs, sums=True)
        b.run()
    for _ in range(3):
        b.out.fill_(-1.0)
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for r, w in zip(b.results, want.results):
            for got, ref in zip(r, w):
                assert torch.equal(got.view(torch.int32), ref.view(torch.int32))
