"""A tensor of the same few whole chunks over and over has their code, whatever their number, and their streams over and over.  So a container of many chunks can be held
against the oracle's of a few."""
import torch

from paper_2508_19263_amd import zc


def assert_few_over_and_over(got, info, few, times):
    """got, info: container (CUDA tensor) and zc.Info of `times` times the chunks of `few`, the oracle's container of them (numpy)."""
    one = zc.validate_container(few)
    n_few = one.n_chunks
    assert info.n_chunks == n_few * times and info.n_fields == one.n_fields
    assert list(info.mode) == list(one.mode) and [bytes(c) for c in info.code_len] == [bytes(c) for c in one.code_len]
    few = torch.from_numpy(few).to(got.device)
    index = lambda t, at, n: t[at:at + 4 * n].view(torch.int32).long()
    at_few, at = one.payload_offset, info.payload_offset
    for f in range(one.n_fields):
        of_all, of_few = index(got, info.index_offset[f], n_few * times + 1), index(few, one.index_offset[f], n_few + 1)
        assert torch.equal(of_all.diff(), of_few.diff().repeat(times)), f
        n = 16 * int(of_few[-1] - of_few[0])
        assert torch.equal(got[at:at + n * times].view(times, n), few[at_few:at_few + n].expand(times, n)), f
        at_few, at = at_few + n, at + n * times
    assert at_few == few.numel() and at == got.numel() == info.total_bytes
