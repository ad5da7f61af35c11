"""Chunk attention where tiles lose their mask: windows around the smallest one that holds a whole tile of 64 (32)
keys for every query of a block, rings that are full, begin in the middle and wrap inside a tile, pages smaller than the
rows a wave brings and larger than a tile, and a global cache of more than 64 pages."""
import math

import numpy as np
import pytest

import paper_2512_17452_amd as wg
from oracle import attend_definition
from test_gpu_prefill_shapes import _feed, _tol

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("d,G", [(128, 4), (128, 8), (64, 4), (64, 1)])
@pytest.mark.parametrize("W,P,tau,chunks", [
    (94, 8, 0.6, [[200, 33], [65, 160], [31, 64]]),
    (95, 16, 0.6, [[129, 64], [96, 300], [64, 1]]),
    (160, 128, 0.3, [[333, 161], [1, 95], [256, 128]]),
    (256, 16, 1.5, [[255, 600], [289, 70], [64, 320]]),     # nothing admitted: windows alone
    (96, 2, 0.0, [[97, 350], [160, 31], [33, 129]]),        # everything admitted, more than 64 pages
])
def test_tiles_inside_all_windows(d, G, W, P, tau, chunks):
    worst = 0.0
    for s, t0, K, V, g, q, out in _feed(wg.BF16, d, G, 2, chunks, W, P, tau, seed=3 * d + G + W):
        ref = attend_definition(K, V, g, q, t0 + np.arange(len(q)), W, tau, 1 / math.sqrt(d))
        assert np.isfinite(out).all(), (s, t0)
        worst = max(worst, np.abs(out - ref).max())
    assert worst <= _tol(wg.BF16, d, G), worst
