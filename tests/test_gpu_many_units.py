"""A launch of odd pairs with more units than HIP launches workgroups for: the
workgroups share them.  The units past the table's are skipped, so the one small
pair's tiles are bitwise iqa_tiles'."""

from __future__ import annotations

import ctypes

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import _lib, iqa_tiles, synth
from paper_2501_10653_amd._lib import IqaPair
from tests.gpu_util import requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]


def test_more_units_than_workgroups():
    N, NT = 450, 45
    lib = _lib.load()
    x, y = (to_dev(a) for a in synth.random_pair(N, np.random.default_rng(3), neg_frac=0.3, scale=1.0))
    c = 1e-6
    want = iqa_tiles(x, y, NT)
    out = torch.full((2, N // NT, N // NT), -1.0, device="cuda")
    pair = IqaPair(x.data_ptr(), y.data_ptr(), N, NT, float(np.float32(c)) / 2.0, c, c, c,
                   out[0].data_ptr(), out[1].data_ptr(), None)
    host, units = np.zeros(_lib.BATCH_DESC_BYTES, np.uint8), ctypes.c_int64()
    assert lib.iqa_odd_batch_describe(ctypes.byref(pair), 1, host.ctypes.data, ctypes.byref(units)) == 0
    table = torch.from_numpy(host).cuda()
    torch.cuda.synchronize()
    for total in (units.value, units.value + (1 << 24)):
        out.fill_(-1.0)
        torch.cuda.synchronize()
        assert lib.iqa_odd_tiles_batched(table.data_ptr(), 1, total, None) == 0
        torch.cuda.synchronize()
        for got, ref in zip(out, (want.lisi, want.auglisi)):
            assert torch.equal(got.view(torch.int32), ref.view(torch.int32)), total
