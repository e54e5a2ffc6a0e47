"""The tuner's table of 1D forms: an entry applies only to the build whose forms it compared."""

import json

import numpy as np
import pytest

from paper_2601_01596_amd import ffcz as F
from tests.test_gpu_batched import _member, _run

pytestmark = pytest.mark.gpu


def _entries(path, lg):
    doc = json.loads(path.read_text())
    return {k: e for k, e in doc["entries"].items() if f" lg={lg} " in k}


def _clear():
    F.ffcz_set_tuning(1, "")
    F.ffcz_clear_tuning()


# work lengths 2^13 and 2^14: below and at the length from which the tiled form is the default
@pytest.mark.parametrize("L,lg", [(4500, 13), (9000, 14)])
@pytest.mark.parametrize("choice", [0, 1])
def test_an_entry_of_other_forms_is_timed_again(tmp_path, L, lg, choice):
    # a table whose entries say "default" or "other" without naming the forms
    import torch
    path = tmp_path / "plans.json"
    arch = torch.cuda.get_device_properties(0).gcnArchName
    old = f"{arch} f32 sig lg={lg} n<=4 kinds=b"
    path.write_text('{\n "format": "ffcz tile plans 1",\n "entries": {\n'
                    f'  "{old}": {{"choice": {choice}, "ms": [1.00000, 2.00000]}}\n }}\n}}\n')
    probs = [_member((L,), 900 + i, np.float32) for i in range(3)]
    try:
        F.ffcz_clear_tuning()
        assert F.ffcz_set_tuning(1, str(path)) == F.OK
        ys, st, _ = _run(probs)
        assert st == F.OK
        timed = {k: e for k, e in _entries(path, lg).items() if k != old}
        assert len(timed) == 1 and len(next(iter(timed.values()))["ms"]) == 2, timed
    finally:
        _clear()


def test_resident_and_streamed_loops_have_their_own_entries(tmp_path):
    path = tmp_path / "plans.json"
    probs = [_member((9000,), 900 + i, np.float32) for i in range(3)]
    try:
        F.ffcz_clear_tuning()
        assert F.ffcz_set_tuning(1, str(path)) == F.OK
        a, sa, _ = _run(probs, resident_1d=1)
        b, sb, _ = _run(probs, resident_1d=0)
        assert sa == F.OK and sb == F.OK
        timed = _entries(path, 14)
        assert len(timed) == 2 and all(len(e["ms"]) == 2 for e in timed.values()), timed
        for y, z in zip(a, b):
            assert np.array_equal(y.view(np.uint8), z.view(np.uint8))
        # a table read back is not timed again
        F.ffcz_clear_tuning()
        assert F.ffcz_set_tuning(1, str(path)) == F.OK
        before = path.read_text()
        _run(probs, resident_1d=1)
        assert path.read_text() == before
    finally:
        _clear()
