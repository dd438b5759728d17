"""Times of decode calls against each other's: which codes a tensor has, what lies beside it and how many tensors there are must not cost what
a wrong table or a wrong loop does.  Every limit lies between what is measured as it should be and as it was when it was not (in the comments);
times are the least of several, on the same data and device."""
import pytest
import torch

from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024
BF16, FP8, BYTES, E5M2 = zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2


def decode_us(xs, fmt, chunk, policy=zc.POLICY_HUFF_ALL):
    b = zc.Batch(xs, [x.numel() for x in xs], zc.params(fmt, chunk, streams=64, policy=policy))
    b.compress()
    b.prepare_outputs()
    b.plan_decompress()
    times = []
    for _ in range(9):
        start, end = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
        start.record()
        for _ in range(8):
            b.run_decompress()
        end.record()
        torch.cuda.synchronize()
        times.append(start.elapsed_time(end) * 125)
    return min(times)


def test_byte_symbol_tensors_beyond_a_compute_unit_each():
    """11 us for 256 and for 300 (19)."""
    x = wl.fp8_weight(4096, DEV, 1)
    a, b = (decode_us([x] * n, BYTES, 256 * KIB, zc.POLICY_AUTO) for n in (256, 300))
    print("us", a, b, flush=True)
    assert b < 1.4 * a
