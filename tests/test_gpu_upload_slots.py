"""Uploads go through a few page-locked buffers in turn.  A call that waits for one waits for that buffer's own transfer: not for what other streams do, and without
a call that a capture elsewhere does not allow."""
import time

import pytest
import torch

from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def cycles_per_second():
    a, b = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
    torch.cuda._sleep(1000)
    a.record()
    torch.cuda._sleep(10 ** 6)
    b.record()
    torch.cuda.synchronize()
    return 10 ** 6 / (a.elapsed_time(b) * 1e-3)


def test_a_call_waits_for_its_buffer_only():
    x = wl.fp8_weight(50000, seed=1).to(DEV)
    b = zc.Batch([x], [x.numel()], zc.params(zc.FMT_FP8_E4M3, 65536))
    b.compress()
    b.decompress()
    busy, other, captured = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    y, z = torch.zeros(64, device=DEV), torch.ones(64, device=DEV)
    speed = cycles_per_second()
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    start = time.perf_counter()
    with torch.cuda.stream(other):
        torch.cuda._sleep(int(4 * speed))                        # what another stream does: four seconds
    with torch.cuda.stream(captured):
        graph.capture_begin(capture_error_mode="relaxed")
        y.add_(z)
    with torch.cuda.stream(busy):
        torch.cuda._sleep(int(1.5 * speed))                      # in front of the uploads: one and a half, then six uploads through four buffers
        for _ in range(6):
            b.plan_decompress()
        waited = time.perf_counter() - start
        b.run_decompress()
    with torch.cuda.stream(captured):
        y.add_(z)
        graph.capture_end()
    assert not other.query() and waited < 3.5, waited
    torch.cuda.synchronize()
    assert 1.2 < waited, waited
    assert torch.equal(b.out[0], x.view(torch.uint8))
    for k in range(3):
        graph.replay()
        torch.cuda.synchronize()
        assert bool((y == 2 * (k + 1)).all())
