"""The chunk index where its scan changes hands: up to 512 chunks a wavefront per field, beyond that passes of 8,192 chunks of the whole
workgroup; two and three fields, both orders, fields whose sizes start at any word.  And one step's pages of tensors of different lengths, some of
them deltas, whose headers come from one.  Whole containers against the oracle's: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def fp8(n, seed):
    rng = np.random.default_rng(seed)
    return ((rng.integers(0, 2, n) << 7) | (np.minimum(rng.geometric(0.4, n), 15) << 3) | rng.integers(0, 8, n)).astype(np.uint8)


@pytest.mark.parametrize("reverse", [0, 1])
@pytest.mark.parametrize("chunks", [1, 3, 511, 512, 513, 8191, 8193, 16389])
def test_index_of_two_fields(chunks, reverse):
    """Two tensors in one call: the second one's sizes lie behind the first one's, which are few and odd."""
    lengths = [3 * 256, (chunks - 1) * 256 + 200]
    xs = [fp8(n, chunks + i) for i, n in enumerate(lengths)]
    print("case", chunks, reverse, flush=True)
    b = zc.Batch([torch.from_numpy(x).to(DEV) for x in xs], lengths, zc.params(zc.FMT_FP8_E4M3, 256, streams=4, flags=zc.FLAG_REVERSE_FIELDS if reverse else 0))
    b.compress()
    for i, x in enumerate(xs):
        want = o.compress(x, lengths[i], o.params(zc.FMT_FP8_E4M3, 256, (0, 0, 0), 4, payload_order=reverse))
        assert np.array_equal(b.container(i).cpu().numpy(), want), i


@pytest.mark.parametrize("reverse", [0, 1])
@pytest.mark.parametrize("chunks", [512, 513])
def test_index_of_three_fields(chunks, reverse):
    n = chunks * 1024
    rng = np.random.default_rng(chunks)
    x, scales = rng.integers(0, 256, n // 2).astype(np.uint8), np.minimum(rng.geometric(0.3, n // 32), 255).astype(np.uint8)
    print("case", chunks, reverse, flush=True)
    want = o.compress(x, n, o.params(zc.FMT_FP4_E2M1_MX, 512, (0, 0, 0), 8, payload_order=reverse), scales=scales)
    got, _ = zc.compress(torch.from_numpy(x).to(DEV), n, zc.params(zc.FMT_FP4_E2M1_MX, 512, streams=8, flags=zc.FLAG_REVERSE_FIELDS if reverse else 0),
                         scales=torch.from_numpy(scales).to(DEV))
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("fmt", [zc.FMT_FP8_E4M3, zc.FMT_BF16])
@pytest.mark.parametrize("reverse", [0, 1])
def test_headers_of_one_code(fmt, reverse):
    per = 1 if fmt == zc.FMT_FP8_E4M3 else 2
    lengths = [n * 2048 for n in (32, 1, 33, 512)]
    xs = [fp8(n * per, i) for i, n in enumerate(lengths)]
    if per == 2:
        xs = [(0.02 * np.random.default_rng(i).standard_normal(n)).astype(np.float32).view(np.uint32) >> 16 for i, n in enumerate(lengths)]
        xs = [x.astype(np.uint16).view(np.uint8) for x in xs]
    base = [np.zeros(n * per, np.uint8) for n in lengths]
    print("case", fmt, reverse, flush=True)
    for bases in (None, base):
        p = zc.params(fmt, 2048 * per, streams=8, flags=zc.FLAG_REVERSE_FIELDS if reverse else 0)
        q = o.params(fmt, 2048 * per, (0, 0, 0), 8, payload_order=reverse)
        on = [torch.from_numpy(x).to(DEV) for x in xs]
        b = zc.Batch(on, lengths, p, xor_bases=[torch.from_numpy(x).to(DEV) for x in bases] if bases else None)
        b.compress(zc.train_code(on[0], lengths[0], p))
        for i, x in enumerate(xs):
            want = o.compress_with_code(x, lengths[i], q, *o.train_code(xs[0], lengths[0], q), **({"xor_base": bases[i]} if bases else {}))
            assert np.array_equal(b.container(i).cpu().numpy(), want), (i, bases is None)
