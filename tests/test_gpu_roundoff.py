"""Roundoff of the accumulation and of the quotient, where a bound is small enough
to see the order of additions.

Sums of a constant image.  A block is at most four quads, each summed in pairs
(exact: doublings), so it has two roundings, of 12c and 16c; the lane's compensated
sum and its fold have one each; sums of equal lanes, waves and parts are doublings
again where their counts are powers of two.  Four units in all.  (A chain over the
32 pixels of eight quads is off by 6 units for the constant below: its offset from
the grid of the partial sums is lost in every addition.)

LISI from the exported sums.  Eq. 1 of them in FP64 against the kernel's value: one
rounding, and terms of second order: 1.01 units.  (Numerator, denominator and
quotient each rounded: up to three.)
"""

from __future__ import annotations

import numpy as np
import pytest
import torch

from paper_2501_10653_amd import iqa_tiles, synth
from tests.gpu_util import rel_errors, requires_gpu, to_dev

pytestmark = [pytest.mark.gpu, requires_gpu]

U = 2.0 ** -24
C = 1.0 + 2.0 ** -20 - 2.0 ** -23


# rows of up to 64 quads in one, four, eight and sixteen waves, batches of four and
# eight, long rows, parts; off: floats off a 16-byte boundary
@pytest.mark.parametrize("N,NT,off", [(2048, 16, 0), (4096, 16, 0), (512, 32, 0), (1024, 32, 0), (2048, 32, 0),
                                      (2048, 64, 0), (1024, 128, 0), (2048, 128, 0), (2048, 256, 0),
                                      (1024, 512, 0), (64, 8, 0), (64, 4, 0), (1024, 64, 1), (2048, 256, 1)])
def test_sums_of_a_constant(N, NT, off):
    buf = torch.full((2, N * N + 4), C, device="cuda")
    x, y = (b[off:off + N * N].view(N, N) for b in buf)
    y *= 0.5
    res = iqa_tiles(x, y, NT, sums=True)
    torch.cuda.synchronize()
    got = res.sums.double().cpu().numpy()
    for k, c in ((2, C), (3, C / 2)):
        assert rel_errors(got[:, k], np.full(len(got), c * NT * NT)).max() <= 4 * U


@pytest.mark.parametrize("N,NT", [(256, 32), (1024, 16), (1024, 64), (2025, 45), (1000, 50), (480, 12), (600, 300),
                                  (1024, 512), (900, 9), (450, 225)])
def test_lisi_of_the_exported_sums(N, NT):
    rng = np.random.default_rng(N + NT)
    x, y = synth.random_pair(N, rng, neg_frac=0.3, nan_frac=0.01, scale=1e-3)
    res = iqa_tiles(to_dev(x), to_dev(y), NT, sums=True)
    torch.cuda.synchronize()
    s = res.sums.double().cpu().numpy()
    c = float(np.float32(1e-6))
    want = (c / 2) * s[:, 0] / (np.maximum(s[:, 2], s[:, 3]) + c)
    assert rel_errors(res.lisi.cpu().numpy().ravel(), want).max() <= 1.01 * U
