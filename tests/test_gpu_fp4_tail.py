"""Encoder and decoder of an FP4 tensor's short last chunk (64 lanes, plainly stored element fields): the oracle's containers, byte
for byte, and from them the original bytes, at the edges of rows of elements and of block scales, alone and in a set.  Whole bytes: exact."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"
CB = 16384                                                      # 32,768 elements: 16 rows


@pytest.mark.parametrize("fmt", [zc.FMT_FP4_E2M1_MX, zc.FMT_FP4_E2M1_NV, zc.FMT_FP4_E2M1_MX_BYTES])
@pytest.mark.parametrize("policy", [zc.POLICY_HUFF_ALL, zc.POLICY_AUTO])
def test_short_last_chunks(fmt, policy):
    rng = np.random.default_rng(5)
    p, po = zc.params(fmt, CB, streams=64, policy=policy), o.params(fmt, CB, streams=64, policy=policy)
    held = []
    for i, n in enumerate((32, 480, 512, 544, 2048, 2080, 2 * 16384, 32768 - 32, 32768 + 32, 32768 + 2048 * 3 + 64, 3 * 32768 - 16384, 5 * 32768 + 16416)):
        src, sc = (wl.nvfp4_weight if fmt == zc.FMT_FP4_E2M1_NV else wl.mxfp4_weight)(1, n, seed=i)
        if i % 3 == 1:
            sc = torch.from_numpy(rng.integers(0, 256, sc.numel()).astype(np.uint8))        # scales with codes of every length
        if i % 3 == 2:
            src = torch.from_numpy(rng.integers(0, 256, src.numel()).astype(np.uint8))
        for base in (None, torch.from_numpy(rng.integers(0, 256, src.numel()).astype(np.uint8))):
            print("case fmt", fmt, "policy", policy, "n", n, "delta", base is not None, flush=True)
            want = o.compress(src.numpy(), n, po, scales=sc.numpy(), xor_base=None if base is None else base.numpy())
            db = None if base is None else base.to(DEV)
            got, _ = zc.compress(src.to(DEV), n, p, scales=sc.to(DEV), xor_base=db)
            assert np.array_equal(got.cpu().numpy(), want)
            c = torch.from_numpy(want).to(DEV)
            out = torch.full((src.numel() + 32,), 0x5A, dtype=torch.uint8, device=DEV)
            sco = torch.full((sc.numel() + 32,), 0x5A, dtype=torch.uint8, device=DEV)
            zc.decompress(c, zc.read_info(c, check_index=True), out=out, scales_out=sco, xor_base=db)
            assert torch.equal(out[:src.numel()].cpu(), src) and torch.equal(sco[:sc.numel()].cpu(), sc)
            assert bool((out[src.numel():] == 0x5A).all()) and bool((sco[sc.numel():] == 0x5A).all())       # nothing behind either
        held.append((src, sc, n))
    b = zc.Batch([s.to(DEV) for s, _, _ in held], [n for _, _, n in held], p, scales=[sc.to(DEV) for _, sc, _ in held])
    b.compress()
    outs = b.decompress()
    for i, (s, sc, n) in enumerate(held):
        assert torch.equal(outs[i][:s.numel()].cpu(), s) and torch.equal(b.scales_out[i][:sc.numel()].cpu(), sc), i
