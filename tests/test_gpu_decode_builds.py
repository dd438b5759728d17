"""The decoders of one round of workgroups over the tables they choose among: exponent codes of at most four, eight and sixteen bits (refill
periods of 8, 4 and 2), sign+mantissa fields flat, raw, constant and table coded with short and with long codes; each with stretches of narrow
and of wide codes (words that come in a period late, or behind a period's first entry), and tensors with one table-decoded field beside others
with two.  Whole bytes: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024
BF16, FP8, BYTES, E5M2 = zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2
# shares of a tensor and how its symbols spread there (scale of a two-sided geometric distribution)
STEADY_NARROW, STEADY_WIDE = ((1.0, 0.7),), ((1.0, 6.0),)
NARROW_THEN_WIDE, WIDE_THEN_NARROW = ((0.4, 0.5), (0.35, 8.0), (0.25, 0.5)), ((0.3, 8.0), (0.7, 0.4))


def symbols(n, bits, spread, rng, most=None):
    """`most`: only that many values."""
    parts = [np.round(rng.laplace(0, w, int(n * share) + 1)).astype(np.int64) for share, w in spread]
    half = (1 << bits) // 2 if most is None else most // 2
    return np.clip(np.concatenate(parts)[:n] + half, 0, 2 * half - 1)


def tensor(fmt, n, seed, spread, sm, most=None):
    """sm: "flat", "const", or the spread of its values."""
    eb, mb = {BF16: (8, 7), E5M2: (5, 2)}.get(fmt, (4, 3))
    rng = np.random.default_rng(seed)
    e = symbols(n, eb, spread, rng, most)
    if sm == "flat":
        s = rng.permutation(np.arange(n) % (2 << mb))
    elif sm == "const":
        s = np.full(n, 5)
    else:
        s = symbols(n, mb + 1, sm[0], rng, sm[1])
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return torch.from_numpy(v.astype(np.uint16).view(np.int16) if fmt == BF16 else v.astype(np.uint8))


SHORT_SM, LONG_SM, FEW_SM, FOUR_BIT_SM = (((1.0, 60.0),), None), (((1.0, 4.0),), None), (((1.0, 20.0),), 60), (((1.0, 2.0),), 10)
KINDS = [(FP8, 16, "flat", None), (FP8, 8, "flat", None), (E5M2, 16, "flat", None), (E5M2, 8, "flat", None), (E5M2, 4, "flat", 14),
         (BF16, 16, "flat", None), (BF16, 16, "const", None), (BF16, 8, "flat", 100), (BF16, 4, "flat", 14), (BF16, 4, "const", 14),
         (BF16, 16, SHORT_SM, None), (BF16, 16, LONG_SM, None), (BF16, 8, FEW_SM, 100), (BF16, 4, FOUR_BIT_SM, 14),
         (BYTES, 16, "flat", None), (BYTES, 8, "flat", 10), (BYTES, 16, LONG_SM, None)]


@pytest.mark.parametrize("fmt,limit,sm,most", KINDS)
def test_narrow_and_wide_codes(fmt, limit, sm, most):
    size = 2 if fmt == BF16 else 1
    for chunk, nbytes in ((96 * KIB, 3 * 96 * KIB + 5 * KIB + 2 * size), (160 * KIB, 160 * KIB)):
        for k, spread in enumerate((STEADY_NARROW, STEADY_WIDE, NARROW_THEN_WIDE, WIDE_THEN_NARROW)):
            n = nbytes // size
            x = tensor(fmt, n, fmt * 1000 + limit * 10 + k, spread, sm, most)
            raw = x.view(torch.uint8).reshape(-1)
            print("case", fmt, limit, sm, most, chunk, k, flush=True)
            sm_limit = 16 if sm in ("flat", "const", SHORT_SM, LONG_SM) else limit
            for policy in (zc.POLICY_HUFF_ALL, zc.POLICY_AUTO):
                comp = torch.from_numpy(o.compress(raw.numpy(), n, o.params(fmt, chunk, (limit, sm_limit, 0), 64, policy))).to(DEV)
                out, _ = zc.decompress(comp, zc.read_info(comp, check_index=True))
                assert torch.equal(out.view(torch.uint8).reshape(-1)[:raw.numel()].cpu(), raw), (policy, chunk, k)


@pytest.mark.parametrize("sm", [SHORT_SM, LONG_SM])
def test_one_table_decoded_field_beside_two(sm):
    """n_rings: two fields, long rings, four chunks to a workgroup."""
    print("case", sm, flush=True)
    chunk = 64 * KIB
    xs = [tensor(BF16, 4096, 1, ((1.0, 2.0),), sm)]
    for k, (most, kind, spread) in enumerate([(None, "flat", NARROW_THEN_WIDE), (None, "const", STEADY_WIDE), (100, "flat", WIDE_THEN_NARROW), (14, "flat", STEADY_WIDE), (None, sm, NARROW_THEN_WIDE)]):
        xs.append(tensor(BF16, 3 * chunk // 2 + 1500 + k, k + 2, spread, kind, most))
    xs = [x.to(DEV) for x in xs]
    b = zc.Batch(xs, [x.numel() for x in xs], zc.params(BF16, chunk, streams=64))
    b.compress()
    b.prepare_outputs()
    plan = b.plan_decompress()
    b.run_decompress()
    for i, x in enumerate(xs):
        raw = x.view(torch.uint8).reshape(-1)
        assert torch.equal(b.out[i][:raw.numel()], raw), i
    assert plan.fast_kernel == 8 and plan.n_rings == 128 + 32 + 4, (plan.fast_kernel, plan.n_rings)


@pytest.mark.parametrize("tensors", [256, 257, 512])
def test_more_byte_symbol_tensors_than_compute_units(tensors):
    print("case", tensors, flush=True)
    kinds = [tensor(BYTES, 4096 + 64 * s, s, spread, "flat").to(DEV) for s, spread in enumerate((STEADY_NARROW, WIDE_THEN_NARROW, ((1.0, 1.2),)))]
    xs = [kinds[i % 3] for i in range(tensors)]
    b = zc.Batch(xs, [x.numel() for x in xs], zc.params(BYTES, 256 * KIB, streams=64, policy=zc.POLICY_AUTO))
    b.compress()
    b.prepare_outputs()
    b.decompress()
    for i, x in enumerate(xs):
        assert torch.equal(b.out[i][:x.numel()], x), i
