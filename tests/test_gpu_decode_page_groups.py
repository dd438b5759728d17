"""BF16 pages where their decoder's workgroups change from four to eight wavefronts (more pages than seven four-wavefront workgroups per compute unit
hold at once, and as many), single tensors, sets and lists, one to several passes, codes of 2, 4 and 8 symbols per refill step (nine equally likely exponents: four bits at most).  Back to the source: exact."""
import numpy as np
import pytest
import torch

from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def tensor(n, spread, seed):
    rng = np.random.default_rng(seed)
    e = 100 + (np.minimum(rng.geometric(1 / spread, n), 100) if spread > 1 else rng.integers(0, 9, n))
    return torch.from_numpy(((rng.integers(0, 2, n) << 15) | (e << 7) | rng.integers(0, 128, n)).astype(np.uint16).view(np.int16)).to(DEV)


@pytest.mark.parametrize("lanes", [4, 8, 16, 32])
@pytest.mark.parametrize("spread,limit", [(0, 0), (3, 8), (12, 0)])
@pytest.mark.parametrize("delta", [False, True])
def test_pages_on_both_sides(lanes, spread, limit, delta):
    chunk = 32 * lanes                                           # two rows a page
    edge = 64 * 7 * 4 * 256 // lanes
    for pages, rest in ((edge, 0), (edge + 1, 7), (3 * edge + 5, 0)):
        print("case", lanes, spread, delta, pages, flush=True)
        n = pages * chunk // 2 + rest
        x = tensor(n, spread, pages)
        base = torch.zeros(n, dtype=torch.int16, device=DEV) if delta else None
        p = zc.params(zc.FMT_BF16, chunk, max_code_len=(limit, 0, 0), streams=lanes, policy=zc.POLICY_AUTO)
        comp, info = zc.compress(x, n, p, xor_base=base)
        out, _ = zc.decompress(comp, info, xor_base=base)
        assert torch.equal(out[:2 * n].view(torch.int16), x)
        ids = torch.randint(0, pages, (edge + 3,), generator=torch.Generator().manual_seed(pages)).to(torch.int32).to(DEV)
        got, _ = zc.decompress_chunks(comp, info, ids, xor_base=base)
        assert torch.equal(got.view(torch.int16).view(-1, chunk // 2), x[:pages * chunk // 2].view(pages, -1)[ids.long()])


def test_sets_of_lists():
    chunk, lanes, pages = 256, 8, 9000
    xs = [tensor(pages * chunk // 2, 3 + i, i) for i in range(8)]
    b = zc.Batch(xs, [x.numel() for x in xs], zc.params(zc.FMT_BF16, chunk, streams=lanes, policy=zc.POLICY_AUTO))
    b.compress()
    for each in (2000, 7169, 9000):                              # 16,000, 57,352 and 72,000 slots: 57,344 is where it changes
        ids = [torch.randperm(pages, generator=torch.Generator().manual_seed(each + i))[:each].to(torch.int32).to(DEV) for i in range(8)]
        b.set_chunk_ids(ids)
        print("case", each, flush=True)
        for x, i, got in zip(xs, ids, b.decompress()):
            assert torch.equal(got.view(torch.int16).view(-1, chunk // 2), x.view(pages, -1)[i.long()])
