"""Compress calls where a launch's shape changes: sixteen and eight wavefronts per chunk (512 chunks and one more, with a short last
one), and sets that go up and come back by the GPU's own reads and stores or by copies (256 KiB and one tensor more, either way).  Whole
containers against the oracle's: exact."""
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


@pytest.mark.parametrize("fmt,delta,reverse,table", [(zc.FMT_BF16, False, False, True), (zc.FMT_BF16, True, False, True), (zc.FMT_BF16, True, True, True), (zc.FMT_BF16, False, True, False),
                                                    (zc.FMT_FP8_E4M3, False, True, False)])
@pytest.mark.parametrize("tensors", [513, 1100])
def test_short_chunks_of_many_tensors(fmt, delta, reverse, table, tensors):
    """Eight wavefronts per chunk: rows fewer and more than they are, sign+mantissa fields table coded (`table`) and not, deltas, reversed fields."""
    print("case", fmt, delta, reverse, table, tensors, flush=True)
    xs, bases, wants = [], [], []
    flags, order = (zc.FLAG_REVERSE_FIELDS, 1) if reverse else (0, 0)
    for i, nbytes in enumerate((1000, 5000, 9 * KIB, 70 * KIB + 14)):
        x = tensor(fmt, nbytes, i)
        if table:
            x = x & ~0x7C                                        # (few mantissas: codes of unequal lengths)
        base = torch.from_numpy(np.random.default_rng(50 + i).permutation(x.numpy())) if delta else None
        xs.append(x), bases.append(base)
        wants.append(o.compress(x.view(torch.uint8).reshape(-1).numpy(), x.numel(), o.params(fmt, 256 * KIB, (0, 0, 0), 64, payload_order=order),
                                **({"xor_base": base.view(torch.uint8).reshape(-1).numpy()} if delta else {})))
    on, under = [x.to(DEV) for x in xs], [b.to(DEV) for b in bases] if delta else None
    at = [i % 4 for i in range(tensors)]
    b = zc.Batch([on[i] for i in at], [xs[i].numel() for i in at], zc.params(fmt, 256 * KIB, streams=64, flags=flags), xor_bases=[under[i] for i in at] if delta else None)
    b.compress()
    for i in range(tensors):
        assert np.array_equal(b.container(i).cpu().numpy(), wants[at[i]]), i


def uploaded(tensors):
    """Bytes a set of tensors of one block and two chunks each sends up: a descriptor of 160 bytes, five work lists of an item of 8, 1 KiB of header."""
    up = lambda n: (n + 255) // 256 * 256
    return up(160 * tensors) + 5 * up(8 * tensors) + 1024 * tensors


@pytest.mark.parametrize("tensors", [1, 8, 100, 213, 214, 256, 257])
def test_sets_and_their_headers(tensors):
    assert uploaded(213) <= 256 * KIB < uploaded(214)
    fmt, cb = zc.FMT_FP8_E4M3, 4 * KIB
    kinds = [tensor(fmt, 5000 + 16 * i, i) for i in range(7)]
    wants = [o.compress(x.numpy(), x.numel(), o.params(fmt, cb, (0, 0, 0), 64)) for x in kinds]
    lengths = [kinds[i % 7].numel() for i in range(tensors)]
    print("case tensors", tensors, flush=True)
    on = [x.to(DEV) for x in kinds]
    b = zc.Batch([on[i % 7] for i in range(tensors)], lengths, zc.params(fmt, cb, streams=64))
    for _ in range(2):
        b.arena.fill_(0x5A)
        sizes = b.compress()
        b.prepare_outputs()
        outs = b.decompress()
        torch.cuda.synchronize()
        for i in range(tensors):
            assert sizes[i] == len(wants[i % 7]), i
            assert np.array_equal(b.container(i).cpu().numpy(), wants[i % 7]), i
            assert torch.equal(outs[i].view(torch.uint8).reshape(-1)[:lengths[i]].cpu(), kinds[i % 7]), i
