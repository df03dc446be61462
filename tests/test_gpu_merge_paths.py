"""Merges by every path (one thread per parent, lanes per parent, one or
several workgroups per parent) against Eq. 1 / Eq. 2 on FP64 totals, and the
pyramid launch against the chain of merges, bitwise.

Tolerance: the contract's 1e-5.  The sums of non-negative terms are off by at
most 2 (Kahan) + 6 + 2 (lanes, waves) + 2 + 6 (runs) units of FP32 roundoff,
the quotients by 3 more: 21 units, 1.3e-6.
"""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, merge_tiles, pyramid, synth
from tests.gpu_util import aug_errors, rel_errors, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]

TOL = 1e-5


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


def level(ns, seed):
    rng = np.random.default_rng(seed)
    s = rng.uniform(0.5, 1.0, (ns * ns, 4)) * np.array([2e3, 1e-3, 4e-2, 4e-2])
    s[rng.uniform(size=ns * ns) < 0.1] = 0.0          # blank tiles
    return s.astype(np.float32)


def check(res, s, ns, f):
    n = ns // f
    t = s.astype(np.float64).reshape(n, f, n, f, 4).sum(axis=(1, 3)).reshape(-1, 4)
    c = float(np.float32(1e-6))
    got = res.sums.double().cpu().numpy()
    for k in range(4):
        assert rel_errors(got[:, k], t[:, k]).max() <= TOL, (ns, f, k)
    lisi = (c / 2) * t[:, 0] / (np.maximum(t[:, 2], t[:, 3]) + c)
    aug = 1.0 - t[:, 1] / (t[:, 2] + t[:, 3] + c)
    assert rel_errors(res.lisi.cpu().numpy().ravel(), lisi).max() <= TOL
    assert aug_errors(res.auglisi.cpu().numpy().ravel(), aug).max() <= TOL


@pytest.mark.parametrize("ns,f", [(1, 1), (5, 1), (2, 2), (66, 2), (3, 3), (20, 4), (35, 5), (49, 7),
                                  (64, 8), (9, 9), (33, 11), (32, 16), (34, 17), (25, 25), (64, 64), (65, 65),
                                  (130, 65), (100, 100), (255, 255), (257, 257), (512, 256),
                                  (600, 600), (2048, 16)])
def test_merge_against_fp64(ns, f):
    s = level(ns, 3 * ns + f)
    d = torch.from_numpy(s).cuda()
    res = merge_tiles(d, f)
    out = [torch.full_like(t, -1.0) for t in res]
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=side):
        cap = merge_tiles(d, f, stream=side)
        for o, t in zip(out, cap):
            o.copy_(t)
    other = torch.from_numpy(level(ns, 5 * ns + f)).cuda()
    torch.cuda.synchronize()
    check(res, s, ns, f)
    for _ in range(3):
        with torch.cuda.stream(side):
            g.replay()
            again = merge_tiles(other, f, stream=side)
        torch.cuda.synchronize()
        assert all(same(a, b) for a, b in zip(out, res))
    ref = merge_tiles(other, f)
    torch.cuda.synchronize()
    assert all(same(a, b) for a, b in zip(again, ref))


@pytest.mark.parametrize("N,NT", [(2, 1), (6, 1), (24, 1), (64, 1), (128, 1), (130, 1), (192, 1),
                                  (256, 1), (384, 3), (512, 4), (100, 20)])
def test_pyramid_is_the_chain_of_merges(N, NT):
    rng = np.random.default_rng(N)
    x, y = synth.random_pair(N, rng, neg_frac=0.3, nan_frac=0.01, scale=1.0)
    xd, yd = to_dev(x), to_dev(y)
    levels = pyramid(xd, yd, NT)
    want = [iqa_tiles(xd, yd, NT, sums=True)]
    while want[-1].lisi.shape[0] % 2 == 0:
        want.append(merge_tiles(want[-1].sums, 2))
    torch.cuda.synchronize()
    assert len(levels) == len(want)
    for a, b in zip(levels, want):
        assert a.lisi.shape == b.lisi.shape and a.sums.shape == b.sums.shape
        assert same(a.lisi, b.lisi) and same(a.auglisi, b.auglisi) and same(a.sums, b.sums)
