"""Times of decode calls against each other's: which codes a tensor has, what lies beside it and how many tensors there are must not cost what
a wrong table or a wrong loop does.  Every limit lies between what is measured as it should be and as it was when it was not (in the comments);
times are the least of several, on the same data and device."""
import numpy as np
import pytest
import torch

from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024
BF16, FP8, BYTES, E5M2 = zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2


def spread(fmt, nbytes, width, sm_width=None):
    """Two-sided geometric exponents (and signs+mantissas) of the given scale."""
    eb, mb = {BF16: (8, 7), E5M2: (5, 2)}.get(fmt, (4, 3))
    n, rng = nbytes // (2 if fmt == BF16 else 1), np.random.default_rng(1)

    def draw(bits, w):
        return np.clip(np.round(rng.laplace(0, w, n)).astype(np.int64) + (1 << bits) // 2, 0, (1 << bits) - 1)
    e = draw(eb, width)
    s = rng.permutation(np.arange(n) % (2 << mb)) if sm_width is None else draw(mb + 1, sm_width)
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return torch.from_numpy(v.astype(np.uint16).view(np.int16) if fmt == BF16 else v.astype(np.uint8)).to(DEV)


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


@pytest.mark.parametrize("fmt,narrow,wide,limit", [
    (FP8, (1.0, None), (4.0, None), 1.3),                        # 72 and 76 us (117)
    (E5M2, (1.0, None), (8.0, None), 1.2),                       # 120 and 84 us (206)
    (BF16, (1.0, None), (40.0, None), 1.25),                     # 63 and 68 us (92)
    (BF16, (1.0, 8.0), (1.0, 60.0), 1.1),                        # 119 and 104 us (150)
    (BF16, (1.0, 8.0), (16.0, 2.0), 1.4),                        # 119 and 117 us (305)
])
def test_wide_codes(fmt, narrow, wide, limit):
    nbytes = 8 * 128 * KIB
    a, b = (decode_us([spread(fmt, nbytes, *w)], fmt, 128 * KIB) for w in (narrow, wide))
    print("case", fmt, narrow, wide, "us", a, b, flush=True)
    assert b < limit * a


def test_codes_of_few_symbols():
    """BF16 exponents with codes of at most eight bits, in pairs: 45 us where longer ones take 63 (64 when one at a time)."""
    a, b = (decode_us([spread(BF16, 8 * 128 * KIB, w)], BF16, 128 * KIB) for w in (1.0, 0.3))
    print("us", a, b, flush=True)
    assert b < 0.9 * a


def test_a_small_tensor_with_two_table_decoded_fields_beside_a_large_one_with_one():
    """117 us either way (173 for the two)."""
    large, small = spread(BF16, 8 << 20, 1.0), spread(BF16, 8192, 1.0, 60.0)
    a, b = decode_us([large], BF16, 256 * KIB), decode_us([large, small], BF16, 256 * KIB)
    print("us", a, b, flush=True)
    assert b < 1.2 * a


def test_byte_symbol_tensors_beyond_a_compute_unit_each():
    """11 us for 256 and for 300 (19)."""
    x = wl.fp8_weight(4096, DEV, 1)
    a, b = (decode_us([x] * n, BYTES, 256 * KIB, zc.POLICY_AUTO) for n in (256, 300))
    print("us", a, b, flush=True)
    assert b < 1.4 * a
