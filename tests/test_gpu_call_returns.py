"""What a call has done when it returns.  Dictionary calls over pages, statistics and training have nothing left on their stream: the container may be read, and
the source, the workspace and the destination may be written, on another stream at once.  Exact against the oracle."""
import numpy as np
import pytest
import torch

from oracle import zc_oracle as o
from paper_2508_19263_amd import workloads as wl
from paper_2508_19263_amd import zc

pytestmark = pytest.mark.gpu
DEV = "cuda:0"


def pages(fmt, n, seed):
    return wl.fp8_weight(n, seed=seed).view(torch.uint8) if fmt == zc.FMT_FP8_E4M3 else wl.bf16_weight(n // 2, seed=seed)


@pytest.mark.parametrize("reverse", [False, True])
@pytest.mark.parametrize("fmt", [zc.FMT_FP8_E4M3, zc.FMT_BF16])
def test_dictionary_calls_over_pages(fmt, reverse):
    streams, chunk = 16, 4096
    # (what does not compress is stored as is: pages whose signs+mantissas are not table coded are the page kernels')
    p = zc.params(fmt, chunk, streams=streams, policy=zc.POLICY_AUTO, flags=zc.FLAG_REVERSE_FIELDS if reverse else 0)
    po = o.params(fmt, chunk, streams=streams, policy=o.POLICY_AUTO, payload_order=1 if reverse else 0)
    a = pages(fmt, 100 * chunk, 1)
    lengths, modes = o.train_code(a.numpy(), a.numel(), po)
    code = zc.train_code(a.to(DEV), a.numel(), p)
    assert torch.cuda.current_stream().query()
    side = torch.cuda.Stream()
    # (512 pages: the most that one workgroup has; 513 with the fields in reverse order: the kernel that goes through them once)
    for n_pages, tensors in ((1, 1), (512, 1), (512, 3), (7, 100), (513, 70)):
        print("case", fmt, reverse, n_pages, tensors, flush=True)
        x = pages(fmt, n_pages * chunk, 2)
        want = torch.from_numpy(o.compress_with_code(x.numpy(), x.numel(), po, lengths, modes))
        b = zc.Batch([x.to(DEV) for _ in range(tensors)], [x.numel()] * tensors, p)
        b.arena.zero_()
        torch.cuda.synchronize()
        sizes = b.compress(code)
        if n_pages <= 512 or reverse:
            assert n_pages > 512 or torch.cuda.current_stream().query()
            with torch.cuda.stream(side):
                got = b.arena.clone()
                b.ws.fill_(0xFF)
                for s in b.srcs:
                    s.zero_()
                b.arena.fill_(0x5A)
            side.synchronize()
            offsets = [t.data_ptr() - b.arena.data_ptr() for t in b.comp]
        else:                                                    # a size pass, a scan and an encoder: the sizes are there, the containers when the stream is
            torch.cuda.synchronize()
            got, offsets = b.arena, [t.data_ptr() - b.arena.data_ptr() for t in b.comp]
        for at, size in zip(offsets, sizes):
            assert size == want.numel() and torch.equal(got[at:at + size].cpu(), want), (n_pages, at)


@pytest.mark.parametrize("n_pages", [300, 2000])
def test_a_destination_that_is_too_small(n_pages):
    """The call that says so has stopped writing to it."""
    chunk = 2048
    p = zc.params(zc.FMT_FP8_E4M3, chunk, streams=8)
    x = pages(zc.FMT_FP8_E4M3, n_pages * chunk, 3).to(DEV)
    code = zc.train_code(x, x.numel(), p)
    whole, _ = zc.compress_with_code(x, x.numel(), p, code)
    for with_code in (True, False):
        dst = torch.zeros(whole.numel() // 2, dtype=torch.uint8, device=DEV)
        torch.cuda.synchronize()
        with pytest.raises(zc.ZcError):
            zc.compress_with_code(x, x.numel(), p, code, dst=dst) if with_code else zc.compress(x, x.numel(), p, dst=dst)
        assert torch.cuda.current_stream().query()
        side = torch.cuda.Stream()
        with torch.cuda.stream(side):
            dst.fill_(0x77)
        torch.cuda.synchronize()
        assert bool((dst == 0x77).all())


@pytest.mark.parametrize("fmt", [zc.FMT_BF16, zc.FMT_FP8_E4M3, zc.FMT_FP4_E2M1_MX])
def test_statistics(fmt):
    n = 1 << 20
    x = torch.from_numpy(np.random.default_rng(4).integers(0, 256, n * zc.elem_bits(fmt) // 8).astype(np.uint8)).to(DEV)
    scales = torch.full((n // 32,), 120, dtype=torch.uint8, device=DEV) if zc.scale_block(fmt) else None
    for chunk, streams in ((65536, 64), (2048, 8)):
        zc.stats(x, n, zc.params(fmt, chunk, streams=streams), scales=scales)
        assert torch.cuda.current_stream().query()
