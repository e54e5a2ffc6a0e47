"""Which passes a 3D field's rounds launch: with planes that fit, the plane pass in place of y-inverse,
last axis and y-forward; elsewhere the separate passes.  And the y lengths and rows that the plane
pass's own tests leave out."""

import numpy as np
import pytest

from oracle import ffcz as O
from paper_2601_01596_amd import ffcz as F
from tests.gpu_util import run_gpu
from tests.test_gpu_parity import _check_fp32, _check_fp64, _problem

pytestmark = pytest.mark.gpu


def _launches(fn):
    F.ffcz_profile_enable(True)
    try:
        F.ffcz_profile_read()
        out = fn()
        return out, {k: n for k, (_, n) in F.ffcz_profile_read().items()}
    finally:
        F.ffcz_profile_enable(False)


# 256 entries along y at the smallest, middle and largest row that fits; 64-entry rows at the other
# y lengths.  Many planes where a plane is large: the rule asks for them.
@pytest.mark.parametrize("dt,shape", [(np.float32, (4, 256, 16)), (np.float32, (64, 256, 64)),
                                      (np.float32, (256, 256, 128)), (np.float64, (2, 256, 16)),
                                      (np.float64, (128, 256, 64)), (np.float64, (64, 256, 32)),
                                      (np.float32, (2, 16, 128)), (np.float32, (8, 64, 128)),
                                      (np.float32, (256, 256, 64)), (np.float64, (64, 32, 128))])
def test_small_planes_take_one_pass(dt, shape):
    p = _problem(shape, 95, dt)
    (y, res), n = _launches(lambda: run_gpu(p.x, p.xb, p.E, p.Delta, p.max_iter, record_viol=True))
    assert n["y_inv"] == 0 and n["y_fwd"] == 1, n
    assert n["z_pass"] == res.stats["rounds"]
    orc = O.correct(p.x, p.xb, p.E, p.Delta, p.max_iter, mu=res.stats["margin_used"])
    (_check_fp64 if dt == np.float64 else _check_fp32)(p, y, res, orc)


@pytest.mark.parametrize("dt,shape,kw", [(np.float32, (8, 256, 64), {}), (np.float32, (4, 8, 64), {}),
                                         (np.float64, (64, 64, 64), {"record_masks": True})])
def test_other_fields_take_separate_passes(dt, shape, kw):
    p = _problem(shape, 96, dt)
    (_, res), n = _launches(lambda: run_gpu(p.x, p.xb, p.E, p.Delta, 3, fixed=True, **kw))
    assert res.stats["rounds"] == 3
    assert n["y_inv"] == 3 and n["y_fwd"] == 4, n


# many planes of rows of 64 entries and more: the separate passes are the faster ones from 1024 planes
# on (512 where an FP32 plane has more than 64 KB and rows of 128)
@pytest.mark.parametrize("dt,shape,one", [(np.float32, (1024, 32, 128), False), (np.float32, (512, 32, 128), True),
                                          (np.float64, (1024, 32, 128), False), (np.float32, (1024, 64, 64), True),
                                          (np.float32, (512, 128, 256), False), (np.float32, (512, 64, 256), True)])
def test_many_planes_of_long_rows_take_separate_passes(dt, shape, one):
    import torch
    g = torch.Generator(device="cuda")
    g.manual_seed(7)
    x = torch.randn(shape, generator=g, device="cuda").to(torch.float32 if dt == np.float32 else torch.float64)
    xb = x + 0.01 * (torch.rand(shape, generator=g, device="cuda").to(x.dtype) - 0.5)
    r, n = _launches(lambda: F.correct(x, xb, 0.005, 0.05 * x.numel() ** 0.5, 2, fixed=True, check=False))
    assert r.stats["rounds"] == 2
    assert n["y_inv"] == (0 if one else 2), n
