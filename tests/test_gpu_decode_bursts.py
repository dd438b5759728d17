"""The decoders with whole tables, where their streams run faster than the pieces a row asks for: stretches of rows of nothing but
long codes (up to a word per lane and period: the rings run dry and are filled at once), beside lanes whose words come late, and
short last chunks; codes from a dictionary, in which those symbols are as rare as can be.  Also the exponent codes of more than eight
bits of FP8 E4M3 (singles instead of pairs), and two table-decoded fields with short and with long sign+mantissa codes.  Whole bytes:
exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024


def values(fmt, n, rng, common_exp, common_sm, stretch):
    """Values of a few common exponents and signs+mantissas; in the stretch (a share of the values) of all others."""
    eb, mb = {zc.FMT_BF16: (8, 7), zc.FMT_FP8_E5M2: (5, 2)}.get(fmt, (4, 3))
    e = np.minimum(rng.geometric(0.5, n) - 1, common_exp - 1)
    s = rng.integers(0, common_sm, n)
    a, b = int(n * stretch[0]), int(n * stretch[1])
    e[a:b] = rng.integers(common_exp, 1 << eb, b - a)
    if common_sm < 2 << mb:
        s[a:b] = rng.integers(common_sm, 2 << mb, b - a)
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return v.astype(np.uint16).view(np.int16) if fmt == zc.FMT_BF16 else v.astype(np.uint8)


@pytest.mark.parametrize("fmt,limits,sm", [
    (zc.FMT_FP8_E4M3, (8, 0, 0), 16), (zc.FMT_FP8_E4M3, (7, 0, 0), 16), (zc.FMT_FP8_E4M3, (12, 0, 0), 16), (zc.FMT_FP8_E4M3, (16, 0, 0), 16),
    (zc.FMT_FP8_E5M2, (16, 0, 0), 8), (zc.FMT_FP8_E5M2, (8, 0, 0), 8),
    (zc.FMT_BF16, (16, 16, 0), 256), (zc.FMT_BF16, (16, 16, 0), 24), (zc.FMT_BF16, (16, 12, 0), 24), (zc.FMT_BF16, (8, 8, 0), 24),
    (zc.FMT_FP8_E4M3_BYTES, (16, 16, 0), 16)])
def test_stretches_of_long_codes(fmt, limits, sm):
    rng = np.random.default_rng(fmt * 100 + limits[0] + sm)
    size = 2 if fmt == zc.FMT_BF16 else 1
    for chunk, nbytes in ((64 * KIB, 5 * 64 * KIB + 20 * KIB + 16 * size), (96 * KIB, 3 * 96 * KIB + 2), (256 * KIB, 256 * KIB)):
        n = nbytes // size
        p = o.params(fmt, chunk, limits, 64)
        train = values(fmt, 1 << 20, rng, 3, sm, (0.5, 0.5))
        lengths, modes = o.train_code(train, train.size, p)
        # all of a chunk but its first rows; some rows in the middle; the end with the short last chunk
        for stretch in ((0.02, 0.3), (0.45, 0.5), (0.8, 1.0)):
            x = torch.from_numpy(values(fmt, n, rng, 3, sm, stretch))
            raw = x.view(torch.uint8).reshape(-1)
            print("case fmt", fmt, "limits", limits, "sm", sm, "chunk", chunk, "bytes", nbytes, "stretch", stretch, flush=True)
            comp = torch.from_numpy(o.compress_with_code(raw.numpy(), n, p, lengths, modes)).to(DEV)
            out, _ = zc.decompress(comp, zc.read_info(comp, check_index=True))
            assert torch.equal(out.view(torch.uint8).reshape(-1)[:raw.numel()].cpu(), raw)
