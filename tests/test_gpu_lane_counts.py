"""Counts of 8-bit symbols per chunk lane: chunks of few symbols, of one, of all and of other ones than their neighbours, whose counts alone are written
where the workspace has room to say which those are.  The container is the same without that room, and decodes to the source: exact."""
import numpy as np
import pytest
import torch

from paper_2508_19263_amd import zc

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
