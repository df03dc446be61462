"""Default launches that split a tile over workgroups without asking their
caller to prepare: eager, captured (no workspace exists or is taken then) and
through the no-allocation entry point, all with the same bits, and within
tolerance of the oracle (the contract's 1e-5; the worst case of the sums is
61 units of FP32 roundoff, 3.6e-6)."""

from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import _lib, default_cfg, iqa_tiles, lisi_tiles, synth
from tests.gpu_util import assert_parity, oracle_for, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


def same(a, b):
    return torch.equal(a.view(torch.int32), b.view(torch.int32))


# one and several tiles; four and eight waves per part, one with odd sides
@pytest.mark.parametrize("N,NT", [(300, 300), (600, 600), (600, 300), (375, 375), (450, 225)])
def test_same_bits_eager_captured_and_without_allocation(N, NT):
    assert default_cfg(N, NT)["ksplit"] > 1
    rng = np.random.default_rng(N + NT)
    x, y = synth.random_pair(N, rng, neg_frac=0.3, nan_frac=0.01, scale=1.0)
    x2, y2 = synth.random_pair(N, rng, neg_frac=0.3, scale=1.0)
    xd, yd, xd2, yd2 = to_dev(x), to_dev(y), to_dev(x2), to_dev(y2)
    ns = N // NT
    out = {"lisi": torch.zeros(ns, ns, device="cuda"), "auglisi": torch.zeros(ns, ns, device="cuda")}
    one = torch.zeros(ns, ns, device="cuda")
    s = torch.cuda.Stream()
    s.wait_stream(torch.cuda.current_stream())
    g = torch.cuda.CUDAGraph()
    with torch.cuda.graph(g, stream=s):        # nothing prepared on this stream
        iqa_tiles(xd, yd, NT, out=out, stream=s)
        lisi_tiles(xd, yd, NT, out=one, stream=s)
    eager = iqa_tiles(xd, yd, NT, sums=True)
    torch.cuda.synchronize()
    assert_parity(eager, oracle_for(x, y, NT), what=f"{N}/{NT}")
    for _ in range(3):
        for t in (*out.values(), one):
            t.fill_(-1.0)
        torch.cuda.synchronize()
        with torch.cuda.stream(s):
            g.replay()
            other = iqa_tiles(xd2, yd2, NT, stream=s)
        torch.cuda.synchronize()
        assert same(out["lisi"], eager.lisi) and same(out["auglisi"], eager.auglisi)
        assert same(one, eager.lisi)
    again = iqa_tiles(xd2, yd2, NT)
    torch.cuda.synchronize()
    assert same(other.lisi, again.lisi) and same(other.auglisi, again.auglisi)
    C = 1e-6
    D = float(np.float32(C)) / 2.0
    lo, ao = torch.zeros(ns, ns, device="cuda"), torch.zeros(ns, ns, device="cuda")
    torch.cuda.synchronize()
    st = _lib.load().iqa_tiles_noalloc(xd.data_ptr(), yd.data_ptr(), N, NT, D, C, C, C,
                                       lo.data_ptr(), ao.data_ptr(), None, None,
                                       ctypes.c_void_p(s.cuda_stream))
    torch.cuda.synchronize()
    assert st == 0 and same(lo, eager.lisi) and same(ao, eager.auglisi)
