"""The 64-lane decoders that look up two symbols at a time: containers of the oracle decode to the original bytes, over the refill
periods, unresolved pairs and long codes, lanes whose every period takes 32 bits, short last chunks, deltas and lists of chunk
ids; in calls of few chunks and (by lists) of more than a thousand, which use another build (FP8 E4M3: another kernel).  FP8 E4M3
comes to these kernels with whole chunks of 96 KiB, or of 32 KiB and a short last one.  Whole bytes: exact."""
import ctypes

import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FORMATS = [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2]


def fields(kind, n, rng, top):
    if kind == "geometric":                                     # codes of 1, 2, 3, ... bits, the longest as long as the limit allows
        return np.minimum(rng.geometric(0.5, n) - 1, top - 1)
    if kind == "wide":                                          # a few short codes and many long ones: pairs seldom fit the index
        return np.where(rng.random(n) < 0.3, 0, rng.integers(0, top, n))
    if kind == "uniform":
        return rng.integers(0, top, n)
    if kind == "lanes":                                         # lanes that only ever see the longest codes, beside lanes of the shortest
        v = np.minimum(rng.geometric(0.5, n) - 1, top - 1)
        return np.where((np.arange(n) // 16) % 64 == 5, top - 1, np.where((np.arange(n) // 16) % 64 == 6, 0, v))
    return np.full(n, 1 % top)


def tensor(fmt, n, exp_kind, sm_kind, seed):
    rng = np.random.default_rng(seed)
    eb, mb = {zc.FMT_BF16: (8, 7), zc.FMT_FP8_E5M2: (5, 2)}.get(fmt, (4, 3))
    e, s = fields(exp_kind, n, rng, 1 << eb), fields(sm_kind, n, rng, 2 << mb)
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return torch.from_numpy(v.astype(np.uint16).view(np.int16) if fmt == zc.FMT_BF16 else v.astype(np.uint8))


def kernel_of(c, info, base):
    """What a plan says decodes the container."""
    t, plan = (zc.Tensor * 1)(), zc.BatchPlan()
    out, ws = torch.empty(info.n_elems * zc.elem_bits(info.format) // 8 + 16, dtype=torch.uint8, device=DEV), torch.empty(1 << 20, dtype=torch.uint8, device=DEV)
    t[0].info, t[0].d_comp, t[0].comp_capacity, t[0].out_bytes, t[0].n_elems = info, c.data_ptr(), c.numel(), c.numel(), info.n_elems
    t[0].d_dst, t[0].d_xor_base = out.data_ptr(), None if base is None else base.data_ptr()
    assert zc.lib().zc_decompress_batch_plan(t, 1, ws.data_ptr(), ws.numel(), ctypes.byref(plan), torch.cuda.current_stream().cuda_stream) == 0
    torch.cuda.synchronize()
    return plan.fast_kernel


def decode(fmt, x, base, cb, tag, L=(0, 0, 0), policy=zc.POLICY_HUFF_ALL, lists=True):
    n = x.numel()
    print("case", tag, "fmt", fmt, "n", n, "chunk", cb, "L", L, "policy", policy, flush=True)
    raw = x.view(torch.uint8).reshape(-1)
    braw = None if base is None else base.view(torch.uint8).reshape(-1)
    c = torch.from_numpy(o.compress(raw.numpy(), n, o.params(fmt, cb, L, 64, policy), xor_base=None if braw is None else braw.numpy())).to(DEV)
    info = zc.read_info(c, check_index=True)
    b = None if base is None else base.to(DEV)
    out = torch.full((raw.numel() + 64,), 0x5A, dtype=torch.uint8, device=DEV)
    info.pairs = kernel_of(c, info, b) in (7, 8)
    zc.decompress(c, info, out=out, xor_base=b)
    assert torch.equal(out[:raw.numel()].cpu(), raw), tag
    assert bool((out[raw.numel():] == 0x5A).all()), tag        # nothing behind the tensor
    if not lists:
        return info
    rng = np.random.default_rng(n)
    for n_ids in (5, 1200):
        ids = rng.integers(0, info.n_chunks + 1, n_ids).astype(np.int32)      # repeated, and some out of range
        got, _ = zc.decompress_chunks(c, info, torch.from_numpy(ids).to(DEV), out=torch.full((n_ids * cb,), 0x5A, dtype=torch.uint8, device=DEV), xor_base=b)
        got = got.cpu().reshape(n_ids, cb)
        for i in list(range(min(n_ids, 40))) + [n_ids - 1]:
            want = raw[int(ids[i]) * cb:(int(ids[i]) + 1) * cb] if ids[i] < info.n_chunks else raw[:0]
            assert torch.equal(got[i][:want.numel()], want) and bool((got[i][want.numel():] == 0x5A).all()), (tag, n_ids, i)
    return info


@pytest.mark.parametrize("fmt", FORMATS)
def test_fields_and_periods(fmt):
    size = 2 if fmt == zc.FMT_BF16 else 1
    limits = {zc.FMT_FP8_E4M3: (4, 6, 8, 12, 16)}.get(fmt, (8, 11, 12, 16))
    cb, chunks = (98304, 2) if fmt == zc.FMT_FP8_E4M3 else (2048, 9)
    kinds = [("geometric", "uniform"), ("geometric", "geometric"), ("wide", "wide"), ("lanes", "lanes"), ("uniform", "geometric"), ("geometric", "constant"),
             ("geometric", "uniform"), ("lanes", "uniform"), ("wide", "uniform")]
    seen = set()
    for i, (e, s) in enumerate(kinds):
        for L in limits:
            n = (chunks * cb + (0, 2, 514, 1024, 1026, 2046, 18, 1008, 1030)[i]) // size
            policy = i & 1 if i < 6 else 1
            info = decode(fmt, tensor(fmt, n, e, s, 100 * i + L), None, cb, "%s/%s" % (e, s), L=(L, L, 0), policy=policy)
            if info.pairs:
                longest = info.max_len[0]
                seen.add((2 if longest > 8 else 4 if longest > 4 else 8, info.mode[1], longest > 14))
    # refill periods and sign+mantissa modes these kernels have decoded, and codes beyond FP8 E4M3's index
    if fmt == zc.FMT_FP8_E4M3:
        assert {(r, m) for r, m, _ in seen} == {(2, zc.MODE_HUFF), (4, zc.MODE_HUFF), (2, zc.MODE_RAW), (4, zc.MODE_RAW)} and any(x[2] for x in seen), seen
    else:
        assert {2, 4} <= {r for r, _, _ in seen}, seen


@pytest.mark.parametrize("fmt", FORMATS)
def test_rows_ends_and_deltas(fmt):
    size = 2 if fmt == zc.FMT_BF16 else 1
    few = fmt == zc.FMT_FP8_E4M3
    for i, nbytes in enumerate((2, 16, 30, 1022, 1024, 1026, 2048, 3 * 1024 + 8, 5 * 1024, 6 * 1024 + 1000, 7 * 1024, 9 * 1024 + 16, 65536 + 2, 3 * 65536 - 2)):
        cb, nbytes = (32768, 32768 + nbytes) if few else (65536, nbytes)
        x, b = tensor(fmt, nbytes // size, "geometric", "uniform", i), tensor(fmt, nbytes // size, "wide", "geometric", i + 50)
        assert decode(fmt, x, None, cb, "rows", lists=False).pairs or not few
        decode(fmt, x, b, cb, "delta", lists=False)
    cb = 98304 if few else 4096
    x, b = tensor(fmt, (2 if few else 20) * cb // size + 9, "geometric", "uniform", 3), tensor(fmt, (2 if few else 20) * cb // size + 9, "geometric", "geometric", 4)
    decode(fmt, x, b, cb, "delta lists")
    # (a delta whose sign+mantissa values stay equally likely: the plain field that FP8 E4M3 needs here)
    assert decode(fmt, x, torch.zeros_like(b), cb, "delta of zeros, lists").pairs or not few
    decode(fmt, x, None, cb + 16 if few else 3088, "chunks of rows and one run")


def test_flat_three_bit_code_of_e5m2():
    # exactly equal counts of the eight sign+mantissa values, every number of whole rows modulo four before the last one
    rng = np.random.default_rng(11)
    for rows in range(6):
        for extra in (0, 16, 200, 1008):
            n = (rows * 1024 + extra) // 8 * 8
            if n == 0:
                continue
            sm = rng.permutation(np.repeat(np.arange(8), n // 8))
            e = np.minimum(rng.geometric(0.4, n) - 1, 31)
            x = torch.from_numpy((((sm >> 2) << 7) | (e << 2) | (sm & 3)).astype(np.uint8))
            info = decode(zc.FMT_FP8_E5M2, x, None, 262144, "flat3 rows %d + %d" % (rows, extra), lists=False)
            if n >= 64:
                assert list(info.code_len[1][:9]) == [3] * 8 + [0]


@pytest.mark.parametrize("fmt", FORMATS)
def test_too_short_a_plain_stream_leaves_its_chunk_alone(fmt):
    # the index says that the last chunk's sign+mantissa stream ends before its rows do: the other chunks decode, that one's place
    # in the output keeps what it held (17 units: E5M2's stream has a word per lane, 16 units, that the decoder never uses)
    size, cb, chunks = (2 if fmt == zc.FMT_BF16 else 1), 98304, 5
    x = tensor(fmt, chunks * cb // size, "geometric", "uniform", 21)
    c = torch.from_numpy(o.compress(x.view(torch.uint8).numpy(), x.numel(), o.params(fmt, cb, (0, 0, 0), 64, zc.POLICY_AUTO))).to(DEV)
    info = zc.read_info(c, check_index=True)
    assert kernel_of(c, info, None) in (7, 8)
    assert info.mode[1] == zc.MODE_RAW or len(set(info.code_len[1][:16 if fmt != zc.FMT_FP8_E5M2 else 8])) == 1
    end = info.index_offset[1] + 4 * chunks
    last = c[end:end + 4].view(torch.int32)
    last -= 17
    out = torch.full((chunks * cb,), 0x5A, dtype=torch.uint8, device=DEV)
    zc.decompress(c, info, out=out)
    got, want = out.cpu(), x.view(torch.uint8).reshape(-1)
    assert torch.equal(got[:-cb], want[:-cb]) and bool((got[-cb:] == 0x5A).all())
