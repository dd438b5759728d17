"""Which kernel decodes a call, by its chunks' number and sizes and how they are spread over tensors, and that the bytes come back
whichever it is.  Whole bytes: exact."""
import numpy as np
import pytest
import torch

from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
KIB = 1024
BF16, FP8, BYTES, E5M2 = zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP8_E4M3_BYTES, zc.FMT_FP8_E5M2
LONG = 64 + 32 + 4                                              # plan.n_rings: one table-decoded field, long rings, four chunks a workgroup


def tensor(fmt, nbytes, seed, longest=12, two=False):
    """Exponents with codes of 1, 2, .. `longest` bits; sign+mantissa values in equal numbers (a flat code), or `two`: like the exponents."""
    if nbytes > 1 << 22:
        return tensor(fmt, 1 << 20, seed, longest, two).repeat((nbytes >> 20) + 1)[:nbytes // (2 if fmt == BF16 else 1)].contiguous()
    n = nbytes // (2 if fmt == BF16 else 1)
    eb, mb = {BF16: (8, 7), E5M2: (5, 2)}.get(fmt, (4, 3))
    rng = np.random.default_rng(seed)
    e = np.minimum(rng.geometric(0.5, n) - 1, min(longest, 1 << eb) - 1)
    s = np.minimum(rng.geometric(0.5, n) - 1, longest - 1) if two else rng.permutation(np.arange(n) % (2 << mb))
    if two:                                                     # (the longest code is there in both fields, however short the tensor)
        e[:longest] = s[-longest:] = np.arange(longest)
    v = ((s >> mb) << (eb + mb)) | (e << mb) | (s & ((1 << mb) - 1))
    return torch.from_numpy(v.astype(np.uint16).view(np.int16) if fmt == BF16 else v.astype(np.uint8)).to(DEV)


def decode_set(xs, p, ids=None, bases=None):
    """The plan, after a check of what it decodes."""
    b = zc.Batch(xs, [x.numel() for x in xs], p, xor_bases=bases)
    b.compress()
    cb = p.chunk_bytes
    if ids is not None:
        b.set_chunk_ids([torch.from_numpy(i.astype(np.int32)).to(DEV) for i in ids])
    else:
        b.prepare_outputs()
    for o in b.out:
        o.fill_(0x5A)
    plan = b.plan_decompress()
    b.run_decompress()
    for i, x in enumerate(xs):
        raw = x.view(torch.uint8).reshape(-1)
        if ids is None:
            assert torch.equal(b.out[i][:raw.numel()], raw), i
            if i == len(xs) - 1:                                # and the same container on its own
                alone, _ = zc.decompress(b.container(i), b.arr[i].info, xor_base=None if bases is None else bases[i])
                assert torch.equal(alone, raw)
        else:
            for k, c in enumerate(ids[i]):
                want = raw[int(c) * cb:(int(c) + 1) * cb]
                assert torch.equal(b.out[i][k * cb:k * cb + want.numel()], want), (i, k)
    return plan


CASES = [
    # format, tensors, bytes of each, chunk: kernel, n_rings, kernel of the second list (only where there is one)
    (BF16, 200, 5000, 256 * KIB, 8, LONG, None),                # one round of workgroups
    (BF16, 300, 5000, 256 * KIB, 8, 64 + 1, None),              # more: rings for the one chunk each has
    (BF16, 300, 4096 + 2048, 4096, 8, 64 + 2, None),
    (BF16, 300, 2 * 2048 + 2, 2048, 8, 64 + 4, None),
    (BF16, 300, 5 * 2048 + 1022, 2048, 8, 64 + 8, None),
    (E5M2, 300, 2 * 4096 + 2048, 4096, 7, 64 + 4, None),
    (BYTES, 400, 4096, 256 * KIB, 8, LONG, None),               # small tables: two workgroups on a compute unit
    (BYTES, 600, 4096, 256 * KIB, 8, 64 + 1, None),
    (BYTES, 1, 1100 * 2048, 2048, 8, 64 + 8, None),
    (BYTES, 1100, 2 * 2048, 2048, 8, 64 + 2, None),
    (BF16, 1100, 2 * 2048, 2048, 6, None, None),                # many tensors of few whole chunks
    (BF16, 800, 3 * 2048, 2048, 6, None, None),
    (E5M2, 1100, 2048, 2048, 9, None, None),
    (E5M2, 800, 4 * 1024, 1024, 9, None, None),
    (E5M2, 1100, 3000, 256 * KIB, 9, None, 1),                  # or of one short one
    (E5M2, 1100, 9000, 256 * KIB, 7, 64 + 1, None),
    (FP8, 1, 20 * 64 * KIB, 64 * KIB, 1, None, None),           # FP8: whole chunks from 96 KiB on,
    (FP8, 1, 20 * 96 * KIB, 96 * KIB, 8, LONG, None),
    (FP8, 2, 20 * 32 * KIB + 16, 32 * KIB, 8, LONG, None),      # from 32 KiB where there is a short one,
    (FP8, 2, 20 * 16 * KIB + 9 * KIB, 16 * KIB, 1, None, 1),
    (FP8, 5, 12 * KIB, 256 * KIB, 1, None, 1),                  # short ones alone from 16 KiB,
    (FP8, 5, 20 * KIB, 256 * KIB, 8, LONG, None),
    (FP8, 300, 20 * KIB, 256 * KIB, 1, None, 1),                # one round of workgroups
    (FP8, 1, 20 * (20 * KIB + 16), 20 * KIB + 16, 8, LONG, None),        # chunks that are not whole rows: as short ones
    (FP8, 1, 20 * (12 * KIB + 16), 12 * KIB + 16, 0, None, 1),
    (E5M2, 1100, 2 * 9232, 9232, 7, 64 + 2, None),
    (BF16, 1100, 2 * 9232, 9232, 8, 64 + 2, None),
    (FP8, 1, 1024 * 96 * KIB + 16, 96 * KIB, 1, None, 1),
    (FP8, 1, 1025 * 32 * KIB + 20 * KIB, 32 * KIB, 1, None, 3),
    (FP8, 100, 12 * 32 * KIB + 20 * KIB, 32 * KIB, 1, None, 3),
    (FP8, 300, 32 * KIB + 20 * KIB, 32 * KIB, 1, None, 1),
]


@pytest.mark.parametrize("fmt,tensors,nbytes,chunk,kernel,rings,second", CASES)
def test_sets(fmt, tensors, nbytes, chunk, kernel, rings, second):
    print("case", fmt, tensors, nbytes, chunk, flush=True)
    kinds = [tensor(fmt, nbytes, s, 6 if fmt == FP8 else 12) for s in range(3)]
    plan = decode_set([kinds[i % 3] for i in range(tensors)], zc.params(fmt, chunk, streams=64, policy=zc.POLICY_AUTO if fmt == BYTES else zc.POLICY_HUFF_ALL))
    assert plan.fast_kernel == kernel and (rings is None or plan.n_rings == rings), (plan.fast_kernel, plan.n_rings)
    assert (plan.n_work > 0) == (second is not None) and (second is None or plan.tail_kernel == second), (plan.n_work, plan.tail_kernel)


@pytest.mark.parametrize("longest", [4, 8, 12])                 # refill periods of 8, 4 and 2
def test_two_table_decoded_fields(longest):
    print("case", longest, flush=True)
    x, w = [tensor(BF16, 2 * 2048, s, longest, two=True) for s in range(3)], torch.zeros(2048, dtype=torch.int16, device=DEV)
    p = zc.params(BF16, 2048, streams=64)
    for tensors, kernel, rings in ((100, 8, 128 + 32 + 4), (600, 8, 128 + 2), (1100, 6, None)):
        plan = decode_set([x[i % 3] for i in range(tensors)], p, bases=[w] * tensors)
        assert plan.fast_kernel == kernel and (rings is None or plan.n_rings == rings), (tensors, plan.fast_kernel, plan.n_rings)


def test_a_few_chunks_more_than_fill_the_gpu_with_two_table_decoded_fields():
    chunk = 128 * KIB
    kinds = [tensor(BF16, 41 * chunk, s, 12, two=True) for s in range(2)]
    p = zc.params(BF16, chunk, streams=64)
    whole = [kinds[i % 2] for i in range(100)]                  # 4,100 chunks
    assert decode_set(whole, p).fast_kernel == 6
    assert decode_set([torch.cat(whole)], p).fast_kernel == 6   # (and one tensor alone)
    for xs, ids in ((whole[:99] + [kinds[0][:kinds[0].numel() - 512]], None), (whole[:99], None), (whole, [np.arange(41) for _ in whole])):
        plan = decode_set(xs, p, ids)
        assert plan.fast_kernel == 8 and plan.n_rings == 128 + 8 and plan.n_work == 0


def test_id_lists_of_fp8():
    for chunk, tail, kernel in ((64 * KIB, 0, 1), (64 * KIB, 20 * KIB, 1), (96 * KIB, 0, 8), (96 * KIB, 1000, 8)):
        print("case", chunk, tail, flush=True)
        x = tensor(FP8, 30 * chunk + tail, 5, 6)
        ids = np.random.default_rng(1).integers(0, 31 if tail else 30, 50)
        ids[7] = 30 if tail else 29
        assert decode_set([x, x], zc.params(FP8, chunk, streams=64), [ids, ids[:9]]).fast_kernel == kernel


@pytest.mark.parametrize("longest", [4, 8, 12])                 # refill periods of 8, 4 and 2
@pytest.mark.parametrize("delta", [False, True])
def test_many_e5m2_tensors_of_few_whole_chunks(longest, delta):
    print("case", longest, delta, flush=True)
    x, w = [tensor(E5M2, 2 * 2048, s, longest) for s in range(3)], torch.zeros(4096, dtype=torch.uint8, device=DEV)
    assert decode_set([x[i % 3] for i in range(1100)], zc.params(E5M2, 2048, streams=64), bases=[w] * 1100 if delta else None).fast_kernel == 9
