"""Calls with masks on FP32 rows of 256 and 512 entries run the direct last-axis pass with the
default plan's formulas: the same bits as the staged tiles, output, masks and gradient."""

import numpy as np
import pytest

from paper_2601_01596_amd import ffcz as F
from paper_2601_01596_amd import workloads as W
from tests.gpu_util import run_gpu

pytestmark = pytest.mark.gpu


# fewer rows than a tile, one tile, several, in 2D and 3D
@pytest.mark.parametrize("shape", [(2, 256), (4, 8, 256), (64, 256), (2, 512), (2, 8, 512), (32, 16, 512),
                                   (64, 64, 256)])
def test_masked_rows_keep_the_staged_bits(shape):
    import torch
    p = W.make_problem("t", W.grf(shape, 2.0, 5), np.float32, 1e-2, 90.0, 200)
    gy = torch.from_numpy(np.random.default_rng(6).standard_normal(shape).astype(np.float32)).cuda()
    K = 4
    out = []
    try:
        for mode in (0, 2):  # 0: the direct form for masks; 2: half tiles, staged
            F.ffcz_set_tuning(mode)
            y, r = run_gpu(p.x, p.xb, p.E, p.Delta, K, fixed=True, record_masks=True)
            yu, _ = run_gpu(p.x, p.xb, p.E, p.Delta, K, fixed=True)
            g = F.correct_backward(gy, r.masks, K).cpu().numpy()
            out.append((y, yu, r.masks.cpu().numpy(), g, r.stats))
    finally:
        F.ffcz_set_tuning(1)
    (y0, u0, m0, g0, s0), (y1, u1, m1, g1, s1) = out
    assert np.array_equal(y0.view(np.uint8), u0.view(np.uint8))  # with masks = without
    assert np.array_equal(y0.view(np.uint8), y1.view(np.uint8))
    assert np.array_equal(m0, m1)
    assert np.array_equal(g0.view(np.uint8), g1.view(np.uint8))
    assert s0 == s1
