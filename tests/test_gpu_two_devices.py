"""A batch of 1D members on a second device, from a thread that has served the first: the library's own
streams are those of the batch's device."""

import numpy as np
import pytest

from paper_2601_01596_amd import ffcz as F
from tests.test_gpu_batched import _check, _member

pytestmark = pytest.mark.gpu


# several length classes, so that lanes and the one-block stream are used; with and without fields
@pytest.mark.parametrize("shapes", [((600,), (9000,), (70000,), (140000,)), ((600,), (70000,), (32, 32))])
def test_batches_follow_their_device(shapes):
    import torch
    if torch.cuda.device_count() < 2:
        pytest.skip("needs two GPUs")
    probs = [_member(s, 950 + i, np.float32) for i, s in enumerate(shapes)]
    for dev in (0, 1):
        mem = [(torch.from_numpy(p.x).cuda(dev), torch.from_numpy(p.xb).cuda(dev), p.E, p.Delta) for p in probs]
        with torch.cuda.device(dev):
            outs, st, stats = F.correct_batched(mem, 200, check=False)
        torch.cuda.synchronize(dev)
        assert st == F.OK
        for p, o, s in zip(probs, outs, stats):
            assert o.device.index == dev
            _check(p, o.cpu().numpy(), s, np.float32)
