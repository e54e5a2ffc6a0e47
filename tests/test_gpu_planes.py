"""The plane pass (y-inverse, last axis and y-forward of a 3D field in one pass, with the check
before it) against the oracle and against the separate passes."""

import numpy as np
import pytest

from oracle import ffcz as O
from paper_2601_01596_amd import ffcz as F
from tests.gpu_util import rel_err, run_gpu
from tests.test_gpu_parity import _check_fp32, _check_fp64, _problem

pytestmark = pytest.mark.gpu


# one column group and several, one row group and several, single-stage transforms along either
# axis (16, 8 and 16 entries), the smallest and the longest of both axes, planes of 2 to 132 KB,
# fewer planes than CUs and more
SHAPES = [(np.float32, (4, 16, 16)), (np.float64, (2, 16, 32)), (np.float64, (8, 32, 16)), (np.float32, (2, 64, 64)),
          (np.float64, (64, 64, 64)), (np.float32, (16, 512, 16)), (np.float32, (4, 16, 512)),
          (np.float64, (4, 16, 256)), (np.float32, (64, 512, 32)), (np.float32, (64, 32, 512)),
          (np.float64, (128, 16, 512)), (np.float64, (128, 512, 32)), (np.float32, (512, 32, 32)),
          (np.float32, (256, 128, 256))]


@pytest.mark.parametrize("dt,shape", SHAPES)
def test_plane_pass_matches_oracle(dt, shape):
    p = _problem(shape, 91, dt)
    y, res = run_gpu(p.x, p.xb, p.E, p.Delta, p.max_iter, record_viol=True)
    orc = O.correct(p.x, p.xb, p.E, p.Delta, p.max_iter, mu=res.stats["margin_used"])
    (_check_fp64 if dt == np.float64 else _check_fp32)(p, y, res, orc)
    if dt == np.float64:
        assert list(res.viol.cpu().numpy()[: orc.rounds + 1]) == orc.viol


@pytest.mark.parametrize("cap,fixed,graph", [(0, False, 1), (1, False, 1), (1, False, 0), (3, True, 1), (200, False, 0)])
def test_plane_pass_round_control(cap, fixed, graph):
    # caps reached before convergence, fixed rounds, and polled chunks in place of posted checks:
    # status, rounds and counts as with the separate passes.  More planes than a chip's worth of
    # blocks: the late ones start after the first has recorded the outcome.
    p = _problem((1024, 64, 64), 92, np.float64)
    out = []
    try:
        for mode in (1, 0):
            F.ffcz_set_tuning(mode)
            y, r = run_gpu(p.x, p.xb, p.E, p.Delta, cap, fixed=fixed, record_viol=True, graph=bool(graph))
            out.append((y, r))
    finally:
        F.ffcz_set_tuning(1)
    (y1, r1), (y0, r0) = out
    assert r1.status == r0.status
    assert np.array_equal(r1.viol.cpu().numpy(), r0.viol.cpu().numpy())
    for k in ("rounds", "converged", "s_clipped_total", "s_guard"):
        assert r1.stats[k] == r0.stats[k], k
    assert rel_err(y1, y0) <= 1e-12


def test_plane_pass_stops_on_nonfinite_input():
    p = _problem((64, 64, 64), 93, np.float32)
    xb = p.xb.copy()
    xb[3, 5, 7] = np.nan
    _, r = run_gpu(p.x, xb, p.E, p.Delta, p.max_iter)
    assert r.status == F.E_NONFINITE
    assert r.stats["nonfinite"] == 1
