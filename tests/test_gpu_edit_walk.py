"""The coding kernels' walk over rows and planes at its edges: rows shorter than, equal to and just
above 32 entries, planes of one row, sets smaller than a flag word, ragged last words, runs and blocks."""

import numpy as np
import pytest

from oracle import edits as ED
from paper_2601_01596_amd import ffcz as F
from paper_2601_01596_amd import workloads as W
from tests.test_gpu_edits import _oracle_encoded

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dt", [np.float32, np.float64])
@pytest.mark.parametrize("shape", [(4,), (64,), (4096,), (16, 2), (2, 4, 2), (8, 4, 32), (2, 2, 64), (64, 2, 64),
                                   (4, 128), (256, 64), (8, 8, 128), (2, 4, 1024), (4, 4096)])
def test_codes_flags_and_expansion(dt, shape):
    # flags and codes equal the oracle's coding of the exported accumulators (integers: exactly), and
    # the decoder's output meets the oracle decoder's at the bars of the other decoder tests
    import torch
    x = (W.grf(shape, 2.0, 31) if len(shape) > 1 else np.random.default_rng(31).standard_normal(shape)).astype(dt)
    E = W.spatial_bound(x, 2e-2)
    xb = W.quantize(x, E).astype(dt)
    D = W.spectral_bound(x, xb, 85.0)
    xt, bt = torch.from_numpy(np.ascontiguousarray(x)).cuda(), torch.from_numpy(np.ascontiguousarray(xb)).cuda()
    enc = F.encode(xt, bt, E, D, 300, export_edits=True, check=False)
    se, fe = enc.spat_edits.cpu().numpy().astype(np.float64), enc.freq_edits.cpu().numpy().astype(np.float64)
    fs, vs = ED.compact(se)
    ff, vf = ED.compact(fe)
    np.testing.assert_array_equal(enc.spat_flags.cpu().numpy(), fs)
    np.testing.assert_array_equal(enc.freq_flags.cpu().numpy(), ff)
    np.testing.assert_array_equal(enc.spat_codes.cpu().numpy(), ED.quantize(vs, enc.step_s))
    np.testing.assert_array_equal(enc.freq_codes.cpu().numpy(), ED.quantize(vf, enc.step_f))
    y = F.decode(bt, enc).cpu().numpy()
    y_orc = ED.decode(xb, _oracle_encoded(enc))
    rel = float(np.max(np.abs(y.astype(np.float64) - y_orc.astype(np.float64)))) / float(np.max(np.abs(y_orc)))
    assert rel <= (1e-12 if dt == np.float64 else 1e-5)
