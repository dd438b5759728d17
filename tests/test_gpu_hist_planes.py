"""Histograms in bit planes: lengths around a run, a row, a round and a part of a block, deltas, every value of a byte, and more than the caches
hold.  Small containers against the oracle's, whole (the code lengths in them follow from the counts); large ones hold one tensor many times over, which leaves its
code as it is.  Exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024


def values(n, seed, spread):
    rng = np.random.default_rng(seed)
    if spread:                                                   # every byte, no two equally often
        return rng.choice(256, n, p=(lambda w: w / w.sum())(1.02 ** rng.permutation(256))).astype(np.uint8)
    return ((rng.integers(0, 2, n) << 7) | (np.minimum(rng.geometric(0.5, n), 15) << 3) | rng.integers(0, 8, n)).astype(np.uint8)


@pytest.mark.parametrize("delta", [False, True])
@pytest.mark.parametrize("fmt", [zc.FMT_FP8_E4M3, zc.FMT_FP8_E5M2, zc.FMT_FP4_E2M1_MX, zc.FMT_FP4_E2M1_NV])
def test_counts_of_ragged_tensors(fmt, delta):
    fp4 = fmt in (zc.FMT_FP4_E2M1_MX, zc.FMT_FP4_E2M1_NV)
    sizes = [16, 32, 4 * KIB - 16, 4 * KIB + 16, 16 * KIB + 16, 48 * KIB, 256 * KIB, 300 * KIB + 32] if fp4 else \
        [1, 15, 17, 4 * KIB - 1, 4 * KIB + 1, 16 * KIB + 3, 48 * KIB, 256 * KIB, 256 * KIB + 1, 300 * KIB + 5]
    for i, nbytes in enumerate(sizes):
        print("case", fmt, delta, nbytes, flush=True)
        n = nbytes * 2 if fp4 else nbytes
        x, base = values(nbytes, i, i % 2), values(nbytes, 100 + i, True) if delta else None
        scales = values(n // zc.scale_block(fmt), 200 + i, i % 2) if fp4 else None
        want = o.compress(x, n, o.params(fmt, 256 * KIB, (0, 0, 0), 64), **({"xor_base": base} if delta else {}), **({"scales": scales} if fp4 else {}))
        on = [None if a is None else torch.from_numpy(a).to(DEV) for a in (x, base, scales)]
        got, _ = zc.compress(on[0], n, zc.params(fmt, 256 * KIB, streams=64), xor_base=on[1], scales=on[2])
        assert np.array_equal(got.cpu().numpy(), want), nbytes


@pytest.mark.parametrize("fmt,chunk,lanes", [(zc.FMT_FP8_E4M3, 256 * KIB, 64), (zc.FMT_FP8_E5M2, 256 * KIB, 64), (zc.FMT_FP8_E4M3, 2 * KIB, 8), (zc.FMT_FP4_E2M1_MX, 256 * KIB, 64)])
@pytest.mark.parametrize("delta", [False, True])
def test_counts_of_large_tensors(fmt, chunk, lanes, delta):
    """275 MiB and a bit (a short last chunk): 1,100 blocks, by lane where chunks are blocks."""
    print("case", fmt, chunk, lanes, delta, flush=True)
    part, copies = 25 * 256 * KIB, 44
    x = torch.from_numpy(values(part, 7, fmt == zc.FMT_FP8_E5M2)).to(DEV)
    base = torch.from_numpy(values(part, 8, False)).to(DEV) if delta else None
    fp4 = fmt == zc.FMT_FP4_E2M1_MX
    per = 2 if fp4 else 1
    scales = torch.from_numpy(values(part * 2 // 32, 9, False)).to(DEV) if fp4 else None
    p = zc.params(fmt, chunk, streams=lanes)
    _, one = zc.compress(x, part * per, p, xor_base=base, scales=scales)
    many = [None if a is None else a.repeat(copies) for a in (x, base, scales)]
    comp, info = zc.compress(many[0], part * copies * per, p, xor_base=many[1], scales=many[2])
    for f in range(info.n_fields):
        assert bytes(info.code_len[f]) == bytes(one.code_len[f]), f
    out, s = zc.decompress(comp, info, xor_base=many[1])
    assert torch.equal(out, many[0]) and (not fp4 or torch.equal(s, many[2]))


@pytest.mark.parametrize("lanes", [4, 8, 16, 32])
@pytest.mark.parametrize("rows", [1, 2, 4, 8, 16])
def test_counts_of_pages(lanes, rows):
    """Counts per (page, lane) pair: tensors that end within a page, in a histogram block of their own and in the middle of one, pages of one value
    (a count of 256 at sixteen rows), deltas; and a workspace without room for the counts."""
    chunk = 16 * rows * lanes
    for i, nbytes in enumerate((chunk, 3 * chunk + 5, 256 * KIB, 256 * KIB + chunk // 2 + 1, 300 * KIB + 7)):
        print("case", lanes, rows, nbytes, flush=True)
        x = values(nbytes, i, False)
        x[nbytes // 2:] = (x[nbytes // 2:] & 0x87) | 0x38         # (one exponent)
        base = values(nbytes, 50 + i, False) if i % 2 else None
        if base is not None:
            base[nbytes // 2:] &= 0x87
        p = zc.params(zc.FMT_FP8_E4M3, chunk, streams=lanes)
        want = o.compress(x, nbytes, o.params(zc.FMT_FP8_E4M3, chunk, (0, 0, 0), lanes), **({} if base is None else {"xor_base": base}))
        on, under = torch.from_numpy(x).to(DEV), None if base is None else torch.from_numpy(base).to(DEV)
        pairs = -(-nbytes // chunk) * lanes
        room = zc.workspace_bytes([nbytes], p)
        for ws_bytes in (room, room - (pairs * 16 + 255) // 256 * 256 - (pairs * 2 + 255) // 256 * 256):
            ws = torch.empty(ws_bytes, dtype=torch.uint8, device=DEV)
            got, _ = zc.compress(on, nbytes, p, xor_base=under, ws=ws)
            assert np.array_equal(got.cpu().numpy(), want), (nbytes, ws_bytes == room)
        with pytest.raises(zc.ZcError):
            zc.compress(on, nbytes, p, xor_base=under, ws=ws[:-256])
