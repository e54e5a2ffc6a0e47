"""1D members at the edges of the length classes: the smallest tiled class, the classes where set-up
and verification turn tiled and the tile width changes, and the longest, each at one signal (fewer
tiles than an XCD group) and at several."""

import numpy as np
import pytest

from paper_2601_01596_amd import ffcz as F
from tests.test_gpu_batched import _check, _member, _run

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("lengths", [(2048,), (1365, 1366), (2730, 2731, 4096), (10922, 10923, 16384),
                                     (21845, 21846, 32768), (131072, 174763), (262144,), (4097, 16385, 65537, 262143)])
def test_class_edges_match_the_oracle(dt, lengths):
    # power-of-two lengths (no chirp) and the longest and shortest of neighbouring Bluestein classes
    probs = [_member((L,), 800 + i, dt) for i, L in enumerate(lengths)]
    ys, st, stats = _run(probs)
    assert st == F.OK, (st, F.ffcz_last_error())
    for p, y, s in zip(probs, ys, stats):
        _check(p, y, s, dt)


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("L", [2730, 2731, 8192, 10923, 16384, 21846])
def test_classes_one_block_and_tiled_same_bits(dt, L):
    probs = [_member((L,), 830 + i, dt) for i in range(3)]
    a, sa, ta = _run(probs, tiled_1d_lg=12)
    b, sb, tb = _run(probs, tiled_1d_lg=21)
    assert sa == F.OK and sb == F.OK
    for x, y, u, v in zip(a, b, ta, tb):
        assert np.array_equal(x.view(np.uint8), y.view(np.uint8))
        assert u == v
