"""Chunks coded by several wavefronts whose bit totals the size pass leaves for the encoder, and (a workspace without room for them) with the encoder adding them
up itself: last rows of one lane, of some and of all, segments of one row and of several, last segments of the last row alone, deltas.  Whole containers against the
oracle's: exact."""
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
        x = (0.02 * rng.standard_normal(nbytes // 2)).astype(np.float32).view(np.uint32) >> 16
        return x.astype(np.uint16) & np.uint16(0xFFC3)                     # (few mantissas: both fields table coded)
    e = np.minimum(rng.geometric(0.4, nbytes), 15 if fmt != zc.FMT_FP8_E5M2 else 31)
    m = 2 if fmt == zc.FMT_FP8_E5M2 else 3
    return ((rng.integers(0, 2, nbytes) << 7) | (e << m) | np.minimum(rng.geometric(0.5, nbytes) - 1, (1 << m) - 1)).astype(np.uint8)


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2])
@pytest.mark.parametrize("delta", [False, True])
def test_totals_left_and_added_up(fmt, delta):
    for i, nbytes in enumerate((2, 16, 1024, 1040, 2046, 17 * KIB, 17 * KIB + 16, 33 * KIB + 1022, 64 * KIB, 5 * 64 * KIB + 48 * KIB + 2)):
        print("case", fmt, delta, nbytes, flush=True)
        x = tensor(fmt, nbytes, i)
        n, base = x.size, tensor(fmt, nbytes, 100 + i) if delta else None
        want = o.compress(x.view(np.uint8), n, o.params(fmt, 64 * KIB, (0, 0, 0), 64), **({"xor_base": base.view(np.uint8)} if delta else {}))
        p = zc.params(fmt, 64 * KIB, streams=64)
        on, under = [None if a is None else torch.from_numpy(a.view(np.int16) if a.dtype == np.uint16 else a).to(DEV) for a in (x, base)]
        room, chunks = zc.workspace_bytes([n], p), -(-nbytes // (64 * KIB))
        for ws_bytes in (room, room - chunks * 16 * 2 * 64 * 4):
            got, _ = zc.compress(on, n, p, xor_base=under, ws=torch.empty(ws_bytes, dtype=torch.uint8, device=DEV))
            assert np.array_equal(got.cpu().numpy(), want), (nbytes, ws_bytes == room)
        with pytest.raises(zc.ZcError):
            zc.compress(on, n, p, xor_base=under, ws=torch.empty(ws_bytes - 256, dtype=torch.uint8, device=DEV))


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2])
@pytest.mark.parametrize("flat", [(True, True), (True, False), (False, True)])
def test_flat_dictionaries(fmt, flat):
    """A dictionary whose limit leaves the flat code as the only one, in both fields and in either (16 bits for the other one), in workspaces full of
    ones where nothing has been left yet, with and without room for the totals: several segments, short last chunks, and one behind whole chunks that other kernels take."""
    limits = tuple((4 if fmt == zc.FMT_FP8_E4M3 else 8) if f else 0 for f in flat) + (0,)
    a = tensor(fmt, 96 * KIB, 7)
    po, p = o.params(fmt, 32 * KIB, limits, 64), zc.params(fmt, 32 * KIB, limits, streams=64)
    lengths, modes = o.train_code(a.view(np.uint8), a.size, po)
    for f in range(2):
        assert (len(set(lengths[f][:16 if fmt == zc.FMT_FP8_E4M3 else 256])) == 1) == flat[f]
    on = lambda x: torch.from_numpy(x.view(np.int16) if x.dtype == np.uint16 else x).to(DEV)
    code = zc.train_code(on(a), a.size, p)
    for i, nbytes in enumerate((1040, 2046, 17 * KIB + 1022, 32 * KIB, 5 * 32 * KIB + 24 * KIB + 2) + ((1030 * 32 * KIB + 5 * KIB + 30,) if flat[0] and flat[1] else ())):
        print("case", fmt, flat, nbytes, flush=True)
        x = np.tile(tensor(fmt, min(nbytes, 32 * KIB), i), -(-nbytes // (32 * KIB)))
        x = x[:nbytes // x.itemsize]
        want = o.compress_with_code(x.view(np.uint8), x.size, po, lengths, modes)
        room, chunks = zc.workspace_bytes([x.size], p), min(-(-nbytes // (32 * KIB)), 1024)
        for ws_bytes in (room, room - chunks * 16 * 2 * 64 * 4):
            got, info = zc.compress_with_code(on(x), x.size, p, code, ws=torch.full((ws_bytes,), 0xFF, dtype=torch.uint8, device=DEV))
            assert np.array_equal(got.cpu().numpy(), want), (nbytes, ws_bytes == room)
        out, _ = zc.decompress(got, info)
        assert np.array_equal(out.cpu().numpy(), x.view(np.uint8)), nbytes
