"""The thread that drives a correction's rounds gives its core to others while it waits long."""

import os
import subprocess
import sys
import threading
import time

import pytest

from paper_2601_01596_amd import ffcz as F

pytestmark = pytest.mark.gpu


def _cpu_seconds(pid):
    with open(f"/proc/{pid}/stat") as f:
        v = f.read().rsplit(")", 1)[1].split()
    return (int(v[11]) + int(v[12])) / os.sysconf("SC_CLK_TCK")


def test_a_long_wait_leaves_the_core_to_others():
    # a busy process and the calling thread on one core: a thread that only spins takes half of it.
    # The call's first check waits for about 0.6 s of copies ahead of it on the stream.
    import torch
    x = torch.randn((64, 64, 64), device="cuda")
    xb = x + 0.01 * (torch.rand((64, 64, 64), device="cuda") - 0.5)
    big = torch.zeros(1 << 30, dtype=torch.uint8, device="cuda")
    other_big = torch.zeros_like(big)

    def load(k):
        for _ in range(k):
            big.copy_(other_big)

    F.correct(x, xb, 0.01, 1.0, 50, check=False)
    load(20)
    torch.cuda.synchronize()
    e0, e1 = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    e0.record()
    load(100)
    e1.record()
    torch.cuda.synchronize()
    copies = int(600.0 / (e0.elapsed_time(e1) / 100))
    core = sorted(os.sched_getaffinity(0))[-1]
    busy = subprocess.Popen([sys.executable, "-c", f"import os; os.sched_setaffinity(0, [{core}])\nwhile True: pass"])
    out = {}
    stream = torch.cuda.current_stream()

    def call():
        os.sched_setaffinity(0, [core])  # this thread only
        with torch.cuda.stream(stream):
            c0, t0, b0 = time.thread_time(), time.perf_counter(), _cpu_seconds(busy.pid)
            r = F.correct(x, xb, 0.01, 1.0, 50, check=False)
            out.update(cpu=time.thread_time() - c0, wall=time.perf_counter() - t0,
                       other=_cpu_seconds(busy.pid) - b0, status=r.status)

    try:
        time.sleep(0.5)
        load(copies)
        t = threading.Thread(target=call)
        t.start()
        t.join()
    finally:
        busy.kill()
        busy.wait()
    print(f"\n[waiting] {out}")
    assert out["status"] == F.OK and out["wall"] > 0.3
    assert out["other"] / (out["other"] + out["cpu"]) >= 0.65
