"""The kernels that give a chunk sixteen wavefronts (64 lanes, two fields): against the oracle at the sizes where a wavefront's
rows begin and end, and beside the kernels with one wavefront per chunk that a call of more chunks uses.  Whole bytes: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
FORMATS = [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2]


def fields(kind, n, rng, top):
    """n symbol values below `top`: one-bit codes (a wavefront's rows then hold less than a word per lane), long codes, all
    values alike often, two values, one value."""
    if kind == "sparse":
        return np.where(rng.random(n) < 0.985, 3 % top, rng.integers(0, top, n))
    if kind == "long":
        return np.minimum(rng.geometric(0.5, n) - 1, top - 1)
    if kind == "uniform":
        return rng.integers(0, top, n)
    if kind == "two":
        return rng.integers(0, 2, n)
    return np.full(n, 1 % top)


def tensor(fmt, n, exp_kind, sm_kind, seed):
    rng = np.random.default_rng(seed)
    eb, mb = {zc.FMT_BF16: (8, 7), zc.FMT_FP8_E5M2: (5, 2)}.get(fmt, (4, 3))
    e, s = fields(exp_kind, n, rng, 1 << eb), fields(sm_kind, n, rng, 2 << mb)
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return torch.from_numpy(v.astype(np.uint16).view(np.int16) if fmt == zc.FMT_BF16 else v.astype(np.uint8))


def check(fmt, x, base, cb, tag, L=(0, 0, 0), order=0):
    print("case", tag, "fmt", fmt, "n", x.numel(), "chunk", cb, "L", L, flush=True)
    n = x.numel()
    p = zc.params(fmt, cb, L, 64, zc.POLICY_HUFF_ALL, flags=zc.FLAG_REVERSE_FIELDS if order else 0)
    po = o.params(fmt, cb, L, 64, zc.POLICY_HUFF_ALL, payload_order=order)
    want = o.compress(x.view(torch.uint8).numpy(), n, po, xor_base=None if base is None else base.view(torch.uint8).numpy())
    comp, info = zc.compress(x.to(DEV), n, p, xor_base=None if base is None else base.to(DEV))
    got = comp.cpu().numpy()
    assert got.shape == want.shape and np.array_equal(got, want), tag
    assert info.total_bytes == len(want)


@pytest.mark.parametrize("fmt", FORMATS)
def test_rows_at_the_wavefronts_edges(fmt):
    size = 2 if fmt == zc.FMT_BF16 else 1
    cb = 32768                                                  # 32 rows: two per wavefront
    for rows, extra in ((0, 1), (0, 17), (1, 0), (2, 16), (15, 1023), (16, 0), (17, 8), (31, 1008), (32, 0), (33, 2), (64 + 18, 514)):
        n = max(1, (rows * 1024 + extra) // size)
        for e, s in (("long", "uniform"), ("sparse", "sparse"), ("sparse", "constant"), ("constant", "long"), ("two", "two")):
            check(fmt, tensor(fmt, n, e, s, rows * 7 + extra), None, cb, "%s/%s rows %d + %d" % (e, s, rows, extra), order=rows & 1)
    # a delta, a limit that makes refill periods of two for every field, and chunks that are not whole rows
    n = (2 * 65536 + 4098) // size
    a, b = tensor(fmt, n, "long", "uniform", 1), tensor(fmt, n, "long", "sparse", 2)
    check(fmt, a, b, 65536, "delta")
    check(fmt, a, None, 65536, "longest codes", L=(15, 15, 0))
    check(fmt, a, None, 40976, "chunks of 40 rows and one run", order=1)


@pytest.mark.parametrize("fmt", FORMATS)
def test_calls_of_many_chunks_write_the_same_containers(fmt):
    # a call of more chunks than the limit goes through the kernels with one wavefront per chunk; its containers are held
    # against those of calls with one tensor each, which do not
    size = 2 if fmt == zc.FMT_BF16 else 1
    for cb in (262144, 32768):
        kinds = [tensor(fmt, (2 * cb + 5 * 1024 + 2 * i) // size, e, s, i).to(DEV)
                 for i, (e, s) in enumerate((("long", "uniform"), ("sparse", "sparse"), ("long", "constant"), ("uniform", "long")))]
        kinds.append((wl.bf16_weight if size == 2 else wl.fp8_e5m2_weight if fmt == zc.FMT_FP8_E5M2 else wl.fp8_weight)(2 * cb // size + 77, DEV, 5))
        p = zc.params(fmt, cb, streams=64)
        single = [zc.compress(x, x.numel(), p)[0].clone() for x in kinds]
        many = [i % len(kinds) for i in range(360)]            # 1,080 chunks
        b = zc.Batch([kinds[k] for k in many], [kinds[k].numel() for k in many], p)
        for i, size_i in enumerate(b.compress()):
            assert size_i == single[many[i]].numel() and torch.equal(b.container(i), single[many[i]]), (cb, i)
        outs = b.decompress()
        for i in range(len(kinds)):
            x = kinds[many[i]].view(torch.uint8).reshape(-1)
            assert torch.equal(outs[i][:x.numel()], x), (cb, i)
