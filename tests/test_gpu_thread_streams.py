"""Two host threads on hipStreamPerThread (one handle, a stream in each thread)
at once: splits by the tuned table, by the built-in rule, and merges of several
runs give the bits of calls made one after the other."""

from __future__ import annotations

import threading

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, merge_tiles, synth
from tests.gpu_util import requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]

PER_THREAD = 2   # hipStreamPerThread


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def test_threads_on_their_own_streams():
    rng = np.random.default_rng(5)
    work = []
    for _ in range(2):
        calls = []
        for N, NT in [(2048, 256), (900, 300), (1024, 512), (450, 225)]:
            x, y = (to_dev(a) for a in synth.random_pair(N, rng, neg_frac=0.3, scale=1.0))
            calls.append(lambda s, x=x, y=y, NT=NT: iqa_tiles(x, y, NT, sums=True, stream=s))
        sums = torch.from_numpy(rng.uniform(0.5, 1.0, (512 * 512, 4)).astype(np.float32)).cuda()
        calls += [lambda s, f=f: merge_tiles(sums, f, stream=s) for f in (512, 256)]
        work.append(calls)
    want = [[c(None) for c in calls] for calls in work]
    torch.cuda.synchronize()
    got, start = [[], []], threading.Barrier(2)

    def run(k):
        start.wait()
        for _ in range(60):
            got[k].append([c(PER_THREAD) for c in work[k]])

    threads = [threading.Thread(target=run, args=(k,)) for k in range(2)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    torch.cuda.synchronize()
    for k in range(2):
        assert len(got[k]) == 60
        for results in got[k]:
            for r, w in zip(results, want[k]):
                assert all(same(a, b) for a, b in zip(r, w))
