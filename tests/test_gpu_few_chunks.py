"""Compress calls where a launch's shape changes: sixteen and eight wavefronts per chunk (512 chunks and one more, with a short last
one), and sets whose headers come back by the GPU's own stores or by a copy (256 KiB of them and one tensor more).  Whole containers
against the oracle's: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024


def tensor(fmt, nbytes, seed):
    rng = np.random.default_rng(seed)
    if fmt == zc.FMT_BF16:
        return torch.from_numpy((0.02 * rng.standard_normal(nbytes // 2)).astype(np.float32)).to(torch.bfloat16).view(torch.int16)
    e = np.minimum(rng.geometric(0.4, nbytes), 15 if fmt != zc.FMT_FP8_E5M2 else 31)
    m = 2 if fmt == zc.FMT_FP8_E5M2 else 3
    return torch.from_numpy(((rng.integers(0, 2, nbytes) << 7) | (e << m) | rng.integers(0, 1 << m, nbytes)).astype(np.uint8))


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2])
@pytest.mark.parametrize("chunks", [512, 513])
def test_wavefronts_per_chunk(fmt, chunks):
    nbytes = (chunks - 1) * 32 * KIB + 20 * KIB + 6
    x = tensor(fmt, nbytes, chunks)
    n = x.numel()
    print("case", fmt, chunks, n, flush=True)
    want = o.compress(x.view(torch.uint8).reshape(-1).numpy(), n, o.params(fmt, 32 * KIB, (0, 0, 0), 64))
    got, _ = zc.compress(x.to(DEV), n, zc.params(fmt, 32 * KIB, streams=64))
    assert np.array_equal(got.cpu().numpy(), want)


@pytest.mark.parametrize("tensors", [1, 256, 257])
def test_sets_and_their_headers(tensors):
    fmt, cb = zc.FMT_FP8_E4M3, 4 * KIB
    xs = [tensor(fmt, 5000 + 16 * (i % 7), i) for i in range(tensors)]
    lengths = [x.numel() for x in xs]
    print("case tensors", tensors, flush=True)
    b = zc.Batch([x.to(DEV) for x in xs], lengths, zc.params(fmt, cb, streams=64))
    for _ in range(2):
        sizes = b.compress()
        b.prepare_outputs()
        outs = b.decompress()
        torch.cuda.synchronize()
        for i, x in enumerate(xs):
            want = o.compress(x.numpy(), lengths[i], o.params(fmt, cb, (0, 0, 0), 64))
            assert sizes[i] == len(want), i
            assert torch.equal(outs[i].view(torch.uint8).reshape(-1)[:x.numel()].cpu(), x), i
