"""Chunks of 512 MiB and more, which are as valid as any multiple of 16 bytes: a tensor of one chunk comes back whole.  The counts
of bits of such a chunk pass 32 bits.  Whole bytes: exact."""
import pytest
import torch

from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
HALF_GIB = 1 << 29


def skewed_bytes(nbytes, mask, seed):
    """Uniform bytes and'ed with other uniform bytes where `mask` has a bit: codes of several lengths for the symbols in those bits."""
    g = torch.Generator(device=DEV)
    g.manual_seed(seed)
    x = torch.randint(0, 256, (nbytes,), generator=g, device=DEV, dtype=torch.uint8)
    for _ in range(2):
        x &= torch.randint(0, 256, (nbytes,), generator=g, device=DEV, dtype=torch.uint8) | (0xFF & ~mask)
    return x


# what the bits are: exponents 0x78 (E4M3), 0x7C (E5M2), a BF16 value's in both bytes; with the sign and mantissa bits skewed as
# well, both fields are table coded (for FP8 in whole symbols that is another kernel, and another again for a short chunk)
@pytest.mark.parametrize("fmt,mask", [(zc.FMT_BF16, 0x7F), (zc.FMT_BF16, 0xFF), (zc.FMT_FP8_E4M3, 0x78), (zc.FMT_FP8_E4M3, 0xFF),
                                      (zc.FMT_FP8_E4M3_BYTES, 0x78), (zc.FMT_FP8_E5M2, 0x7C), (zc.FMT_FP8_E5M2, 0xFF)])
@pytest.mark.parametrize("chunk", [HALF_GIB, HALF_GIB + HALF_GIB // 2])
def test_one_chunk_of_two_fields(fmt, mask, chunk):
    print("case fmt", fmt, "mask", hex(mask), "chunk", chunk, flush=True)
    x = skewed_bytes(HALF_GIB, mask, 3)
    n = x.numel() * 8 // zc.elem_bits(fmt)
    c, info = zc.compress(x, n, zc.params(fmt, chunk, streams=64))
    assert info.n_chunks == 1 and info.total_bytes < x.numel() + (1 << 20)
    out = torch.full((x.numel() + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    zc.decompress(c, info, out=out)
    assert torch.equal(out[:x.numel()], x) and bool((out[x.numel():] == 0x5A).all())


def test_one_chunk_of_fp4():
    x, sc = skewed_bytes(HALF_GIB, 0, 4), skewed_bytes(HALF_GIB * 2 // 32, 0x7F, 5)
    c, info = zc.compress(x, x.numel() * 2, zc.params(zc.FMT_FP4_E2M1_MX, HALF_GIB, streams=64), scales=sc)
    assert info.n_chunks == 1
    out, scales = (torch.full((t.numel() + 64,), 0x5A, dtype=torch.uint8, device=DEV) for t in (x, sc))
    zc.decompress(c, info, out=out, scales_out=scales)
    for got, want in ((out, x), (scales, sc)):
        assert torch.equal(got[:want.numel()], want) and bool((got[want.numel():] == 0x5A).all())


def test_a_stream_of_more_than_2_gib_is_written():
    # a dictionary whose longest code, all ones, is fifteen bits long, over a chunk of 1.25 GiB that has nothing but that symbol
    n = 5 * HALF_GIB // 2
    e = torch.zeros(1 << 16, dtype=torch.uint8)
    for s in range(1, 16):                                      # symbol s half as often as s - 1
        e[: 1 << (16 - s)] = s
    e[0] = 15
    p = zc.params(zc.FMT_FP8_E4M3, n, (15, 4, 0), streams=64)
    code = zc.train_code((e << 3).to(DEV), e.numel(), p)
    assert max(code.code_len[0]) == 15 and code.code_len[0][15] == 15
    x = torch.full((n,), 15 << 3, dtype=torch.uint8, device=DEV)
    dst = torch.full((zc.compress_bound(n, p),), 0x5A, dtype=torch.uint8, device=DEV)
    c, info = zc.compress_with_code(x, n, p, code, dst=dst)
    stream = c[info.payload_offset:info.payload_offset + (n // 8 * 15)]
    assert info.n_chunks == 1 and stream.numel() > 1 << 31
    # every word of the stream but the last ones of its 64 lanes is full of ones
    written = bool((stream[:-4096] == 0xFF).all())
    assert written
