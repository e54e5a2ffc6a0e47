"""Shell sums and bounds at the edges of their kernels: integer shells at the largest |k|, fewer
entries than a block, more block partials than slices, and bound pairs on rows of 2 to 2049."""

import numpy as np
import pytest

from oracle import bounds as B
from paper_2601_01596_amd import ffcz as F
from paper_2601_01596_amd import workloads as W

pytestmark = pytest.mark.gpu


# tolerance: the shell sums run in FP64 in another order, M 2^-53 at most of the sum of M terms of
# one sign; |k| <= 2509 and M < 2^23 here, so 1e-9 of the bound at the very most; 1e-11 leaves the
# transforms' own rounding room
@pytest.mark.parametrize("shape", [(2,), (4,), (4096,), (2, 2), (4, 4096), (1024, 4), (2, 4, 2), (64, 2, 4),
                                   (4, 8, 1024), (256, 512, 2), (64, 64, 64)])
def test_shell_bounds_at_the_edges(shape):
    import torch
    x = np.random.default_rng(41).standard_normal(shape) + 0.25
    d = F.power_spectrum_bounds(torch.from_numpy(x).cuda(), 1e-3).cpu().numpy()
    ref = B.power_spectrum_bounds(x, 1e-3)
    assert d.shape == ref.shape
    assert float(np.max(np.abs(d - ref) / ref)) <= 1e-11


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(16, 2), (8, 4, 4), (4, 4096), (2, 2, 1024)])
def test_bound_pairs_keep_every_entry(dt, shape):
    # arrays that all hold one value give the scalar bound's correction: every pair, the last
    # column and the padding after it included, is in place
    import torch
    x = W.grf(shape, 2.0, 43).astype(dt)
    p = W.make_problem("t", x, dt, 1e-2, 90.0, 50)
    xt, bt = torch.from_numpy(np.ascontiguousarray(p.x)).cuda(), torch.from_numpy(np.ascontiguousarray(p.xb)).cuda()
    D = float(np.dtype(dt).type(p.Delta))
    arr = torch.full(F.half_shape(shape), D, dtype=xt.dtype, device="cuda")
    ra = F.correct_bounds(xt, bt, 50, eps_s=p.E, D_re=arr, check=False)
    rs = F.correct_bounds(xt, bt, 50, eps_s=p.E, delta_f=D, check=False)
    assert ra.status == rs.status
    assert torch.equal(ra.y, rs.y)
