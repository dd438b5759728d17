"""Counts of 8-bit symbols per chunk lane: chunks of few symbols, of one, of all and of other ones than their neighbours, whose counts alone are written
where the workspace has room to say which those are.  The container is the same without that room, and decodes to the source: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc
from tiled import assert_few_over_and_over

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CHUNK = 256 * 1024


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3_BYTES])
@pytest.mark.parametrize("delta", [False, True])
def test_symbols_a_chunk_does_not_have(fmt, delta):
    print("case", fmt, delta, flush=True)
    rng = np.random.default_rng(fmt)
    kinds = []
    for k in range(6):                                           # chunks of random bytes, of few values, of one value, of ranges of their own
        x = rng.integers(0, 256, CHUNK)
        kinds.append(torch.from_numpy((x if k == 0 else x & 0x24 if k == 1 else x * 0 + 77 if k == 2 else 40 * k + x % 30).astype(np.uint8)))
    chunks = 790
    x = torch.cat([kinds[i] for i in rng.integers(0, 6, chunks)] + [kinds[0][:1030]]).to(DEV)
    base = x.roll(CHUNK) if delta else None
    n = x.numel() // (2 if fmt == zc.FMT_BF16 else 1)
    p = zc.params(fmt, CHUNK, streams=64)
    room = zc.workspace_bytes([n], p)
    got = []
    for ws_bytes in (room, room - (chunks + 1) * 8192):
        comp, info = zc.compress(x, n, p, xor_base=base, ws=torch.empty(ws_bytes, dtype=torch.uint8, device=DEV))
        got.append(comp.clone())
    assert torch.equal(got[0], got[1])
    out, _ = zc.decompress(got[0], info, xor_base=base)
    assert torch.equal(out, x)


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3_BYTES])
@pytest.mark.parametrize("delta", [False, True])
def test_streams_of_such_chunks(fmt, delta):
    """Ten such chunks 79 times over (as many as it takes for their symbols to be counted per lane), with and without room for what says which symbols a chunk has: exact against
    the oracle's ten."""
    print("case", fmt, delta, flush=True)
    rng = np.random.default_rng(10 + fmt)
    few = np.concatenate([(x if k == 0 else x & 0x24 if k == 1 else x * 0 + 77 if k == 2 else 20 * k + x % 25).astype(np.uint8) for k, x in
                          enumerate(rng.integers(0, 256, (10, CHUNK)))])
    base = np.roll(few, CHUNK) if delta else None
    per, times = (2 if fmt == zc.FMT_BF16 else 1), 79
    want = o.compress(few, few.size // per, o.params(fmt, CHUNK, (0, 0, 0), 64), xor_base=base)
    x, under = [None if a is None else torch.from_numpy(a).to(DEV).repeat(times) for a in (few, base)]
    n, p = x.numel() // per, zc.params(fmt, CHUNK, streams=64)
    room = zc.workspace_bytes([n], p)
    for ws_bytes in (room, room - 10 * times * 8192):
        got, info = zc.compress(x, n, p, xor_base=under, ws=torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device=DEV))
        assert_few_over_and_over(got, info, want, times)
