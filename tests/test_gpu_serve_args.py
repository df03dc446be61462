"""A server batch on both sides of what the kernel arguments hold (16 and 31
descriptors): every request bitwise its single launch, whichever form carried it."""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, synth
from paper_2501_10653_amd.serve import Server, serve_cfg
from tests.gpu_util import assert_parity, oracle_for, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


@pytest.mark.parametrize("count", [16, 17, 30, 31, 32, 33])
def test_served_in_one_batch(count):
    rng = np.random.default_rng(count)
    shapes = [(128, 32), (256, 64), (384, 128), (96, 12)]
    host = [synth.random_pair(N, rng, neg_frac=0.3, scale=1.0) for N, _ in shapes]
    dev = [(to_dev(x), to_dev(y)) for x, y in host]
    want = [iqa_tiles(x, y, NT, sums=True, cfg=serve_cfg(N, NT))
            for (x, y), (N, NT) in zip(dev, shapes)]
    torch.cuda.synchronize()
    for (x, y), (N, NT), w in zip(host, shapes, want):
        assert_parity(w, oracle_for(x, y, NT), what=f"{N}/{NT}")
    with Server(1 << 30) as srv:
        refs = [srv.add_reference(y) for _, y in dev]
        reqs = [srv.request(dev[i % 4][0], refs[i % 4], shapes[i % 4][1], sums=True)
                for i in range(count)]
        srv.submit(reqs)
        srv.drain()
        assert all(c["status"] == 0 for c in srv.poll())
        assert srv.stats()["max_batch"] == count
    for i, r in enumerate(reqs):
        for k in ("lisi", "auglisi", "sums"):
            got, exp = getattr(r, k), getattr(want[i % 4], k)
            assert torch.equal(got.view(torch.int32), exp.view(torch.int32)), (i, k)
