"""Calls on a stream that is being captured: fixed rounds without statistics are recorded and replay
like the eager call; a loop that waits for its checks is refused at once, not waited for."""

import os
import subprocess
import sys

import pytest

from paper_2601_01596_amd import ffcz as F

pytestmark = pytest.mark.gpu


# the plane pass, separate passes in 3D and 2D, direct rows
@pytest.mark.parametrize("shape,dtype", [((64, 64, 64), "float64"), ((8, 256, 64), "float32"), ((256, 256), "float32"),
                                         ((16, 16, 512), "float32")])
def test_fixed_rounds_replay_like_the_eager_call(shape, dtype):
    import torch
    dt, rounds = getattr(torch, dtype), 5
    code = F.F32 if dt == torch.float32 else F.F64
    g = torch.Generator(device="cuda")
    g.manual_seed(5)

    def noise():
        return 0.01 * (torch.rand(shape, generator=g, device="cuda").to(dt) - 0.5)

    x = torch.randn(shape, generator=g, device="cuda").to(dt)
    xb, y = x + noise(), torch.empty_like(x)
    ws = F.workspace(code, shape, rounds, x.device)
    o = F.ffcz_default_options()
    o.fixed_iterations, o.verify_fp64 = 1, 0

    def call():
        st = F.ffcz_correct(code, shape, x.data_ptr(), xb.data_ptr(), y.data_ptr(), 0.005, 0.02 * x.numel() ** 0.5,
                            rounds, o, ws.data_ptr(), ws.numel(), torch.cuda.current_stream().cuda_stream, None)
        assert st == F.OK, F.ffcz_last_error()

    call()
    torch.cuda.synchronize()
    s = torch.cuda.Stream()
    with torch.cuda.stream(s):
        call()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph, stream=s):
        call()
    for i in range(4):
        xb.copy_(x + noise())
        y.zero_()
        ws.fill_(i)
        torch.cuda.synchronize()
        graph.replay()
        torch.cuda.synchronize()
        replayed = y.clone()
        call()
        torch.cuda.synchronize()
        assert torch.equal(replayed, y), i


CODE = """
import sys, torch
from paper_2601_01596_amd import ffcz as F
def member(shape):
    x = torch.randn(shape, device="cuda")
    return (x, x + 0.01 * (torch.rand(shape, device="cuda") - 0.5), 0.005, 0.02 * x.numel() ** 0.5)
m = {"field": (64, 64, 64), "signals": (9000,)}[sys.argv[1]]
a = member(m)
if sys.argv[1] == "field":
    ws = F.workspace(F.F32, m, 50, a[0].device)
    call = lambda: F.correct(*a, 50, margin=1e-3, ws=ws, check=False).status
else:
    ws, outs = F.batched_workspace([a], 50), [torch.empty_like(a[0])]
    call = lambda: F.correct_batched([a], 50, margin=1e-3, ws=ws, outs=outs, check=False, tiled_1d_lg=12)[1]
s = torch.cuda.Stream()
with torch.cuda.stream(s):
    assert call() == F.OK  # and the words to post to exist
torch.cuda.synchronize()
graph, status = torch.cuda.CUDAGraph(), None
try:
    with torch.cuda.graph(graph, stream=s):
        status = call()
except RuntimeError as e:
    print("capture ended:", str(e).splitlines()[0])
print("status", status)
"""


@pytest.mark.parametrize("kind", ["field", "signals"])
def test_a_loop_that_waits_is_refused_under_capture(kind):
    root = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))
    r = subprocess.run([sys.executable, "-c", CODE, kind], cwd=root, capture_output=True, text=True, timeout=100)
    assert f"status {F.E_HIP}" in r.stdout and "capture ended" in r.stdout, r.stdout + r.stderr
