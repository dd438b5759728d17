"""Whole FP4 chunks whose rows are dealt out to several workgroups: chunks of fewer rows than wavefronts and of many, scale streams of part of a
row to several rows, scales of one value, of few and of nearly all, element fields that are stored plainly and (few values) that are not, deltas.  Whole containers against the oracle's, and
back: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc
from tiled import assert_few_over_and_over

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024


@pytest.mark.parametrize("policy", [zc.POLICY_HUFF_ALL, zc.POLICY_AUTO])
@pytest.mark.parametrize("chunk", [1, 3, 16, 64, 256])
@pytest.mark.parametrize("fmt", [zc.FMT_FP4_E2M1_MX, zc.FMT_FP4_E2M1_NV, zc.FMT_FP4_E2M1_MX_BYTES])
def test_whole_chunks(fmt, chunk, policy):
    rng = np.random.default_rng(chunk)
    for values, spread, delta in ((16, 1, False), (16, 6, True), (16, 120, False), (3, 3, False)):
        nbytes = 5 * chunk * KIB + (chunk * KIB // 2)
        n = nbytes * 2
        print("case", fmt, chunk, policy, values, spread, delta, flush=True)
        x = (rng.integers(0, values, nbytes) | rng.integers(0, values, nbytes) << 4).astype(np.uint8)
        base = rng.integers(0, 256, nbytes).astype(np.uint8) if delta else None
        scales = (100 + np.minimum(rng.geometric(1 / spread, n // zc.scale_block(fmt)), 155)).astype(np.uint8)
        kw = {"xor_base": base} if delta else {}
        want = o.compress(x, n, o.params(fmt, chunk * KIB, (0, 0, 0), 64, policy=o.POLICY_AUTO if policy == zc.POLICY_AUTO else o.POLICY_HUFF_ALL), scales=scales, **kw)
        on = [None if a is None else torch.from_numpy(a).to(DEV) for a in (x, base, scales)]
        got, info = zc.compress(on[0], n, zc.params(fmt, chunk * KIB, streams=64, policy=policy), xor_base=on[1], scales=on[2])
        assert np.array_equal(got.cpu().numpy(), want), (values, spread)
        out, s = zc.decompress(got, info, xor_base=on[1])
        assert torch.equal(out, on[0]) and torch.equal(s, on[2])


@pytest.mark.parametrize("fmt", [zc.FMT_FP4_E2M1_MX, zc.FMT_FP4_E2M1_NV])
@pytest.mark.parametrize("chunk", [2, 4, 16, 33])
def test_many_chunks_decode(fmt, chunk):
    """On both sides of 1,024 chunks, from which NVFP4's scales have workgroups of their own; one tensor and a set."""
    rng = np.random.default_rng(chunk)
    p = zc.params(fmt, chunk * KIB, streams=64)
    for chunks in (1024, 1025, 1700):
        print("case", fmt, chunk, chunks, flush=True)
        nbytes = chunks * chunk * KIB
        x = torch.from_numpy(rng.integers(0, 256, nbytes).astype(np.uint8)).to(DEV)
        scales = torch.from_numpy((100 + np.minimum(rng.geometric(0.3, 2 * nbytes // zc.scale_block(fmt)), 155)).astype(np.uint8)).to(DEV)
        comp, info = zc.compress(x, 2 * nbytes, p, scales=scales)
        out, s = zc.decompress(comp, info)
        assert torch.equal(out, x) and torch.equal(s, scales)
        half = nbytes // 2 // (chunk * KIB) * (chunk * KIB)
        per = zc.scale_block(fmt) // 2
        b = zc.Batch([x[:half], x[half:]], [2 * half, 2 * (nbytes - half)], p, scales=[scales[:half // per], scales[half // per:].clone()])
        b.compress()
        a, c = b.decompress()
        assert torch.equal(a, x[:half]) and torch.equal(c, x[half:])
        assert torch.equal(torch.cat(b.scales_out), scales)


def test_more_chunks_than_a_launch_of_nine_workgroups_each_holds():
    """1,900,000 chunks of 1 KiB, a thousand of them over and over, so that the code is that of the thousand and so is every stream: the thousand against the oracle, the rest
    against the thousand.  (HIP launches fewer than 2^32 threads: 1,864,135 chunks at nine workgroups of 256.)"""
    rng = np.random.default_rng(5)
    fmt, few, times = zc.FMT_FP4_E2M1_MX, 1000, 1900
    x = rng.integers(0, 256, few * KIB).astype(np.uint8)
    scales = (100 + np.minimum(rng.geometric(0.3, 2 * x.size // 32), 155)).astype(np.uint8)
    small = o.compress(x, 2 * x.size, o.params(fmt, KIB, (0, 0, 0), 64), scales=scales)
    p = zc.params(fmt, KIB, streams=64)
    on = [torch.from_numpy(a).to(DEV).repeat(times) for a in (x, scales)]
    got, info = zc.compress(on[0], 2 * on[0].numel(), p, scales=on[1])
    assert_few_over_and_over(got, info, small, times)
    out, s = zc.decompress(got, info)
    assert torch.equal(out, on[0]) and torch.equal(s, on[1])
