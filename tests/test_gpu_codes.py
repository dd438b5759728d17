"""Codes built on the device where their construction changes: alphabets around 32 and 64 symbols (one wavefront's rows, steps of the searches) up to all
256, equal, nearly equal and steeply falling counts, limits that bind at once, later and not at all, weights of more than 32 bits.  Containers against the
oracle's; exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def field(n, symbols, shape, seed):
    """n symbols out of so many, each at least once, under a random renaming."""
    rng = np.random.default_rng(seed)
    if shape == "equal":
        x = np.arange(n) % symbols
    elif shape == "near":
        x = np.concatenate([np.arange(symbols), rng.integers(0, symbols, n - symbols)])
    else:
        w = 0.7 ** np.arange(symbols)
        x = np.concatenate([np.arange(symbols), rng.choice(symbols, n - symbols, p=w / w.sum())])
    return rng.permutation(256)[:symbols][x].astype(np.uint16)


@pytest.mark.parametrize("symbols", [2, 3, 16, 31, 32, 33, 63, 64, 65, 127, 128, 129, 255, 256])
@pytest.mark.parametrize("limit", [0, 8, 9, 11])
def test_alphabets(symbols, limit):
    n = 40000
    for i, shape in enumerate(("equal", "near", "steep")):
        print("case", symbols, limit, shape, flush=True)
        e, m = field(n, symbols, shape, i), field(n, symbols, ("steep", "equal", "near")[i], 10 + i)
        x = (((m >> 7) << 15) | (e << 7) | (m & 127)).astype(np.uint16)
        want = o.compress(x.view(np.uint8), n, o.params(zc.FMT_BF16, 65536, (limit, limit, 0), 64))
        got, _ = zc.compress(torch.from_numpy(x.view(np.int16)).to(DEV), n, zc.params(zc.FMT_BF16, 65536, max_code_len=(limit, limit, 0), streams=64))
        assert np.array_equal(got.cpu().numpy(), want), shape


@pytest.mark.parametrize("symbols", [20, 50, 256])
def test_weights_beyond_32_bits(symbols):
    """One tensor 6,800 times over: 16 times its symbols are more than 2^32, and its code stays what it is."""
    n, copies = 40000, 6800
    x = ((field(n, symbols, "steep", 3) << 7) | (field(n, min(symbols, 128), "near", 4) % 128)).astype(np.uint16)
    one = torch.from_numpy(x.view(np.int16)).to(DEV)
    p = zc.params(zc.FMT_BF16, 262144, streams=64)
    _, a = zc.compress(one, n, p)
    many = one.repeat(copies)
    comp, b = zc.compress(many, n * copies, p)
    for f in range(2):
        assert bytes(a.code_len[f]) == bytes(b.code_len[f]), f
    out, _ = zc.decompress(comp, b)
    assert torch.equal(out.view(torch.int16), many)
