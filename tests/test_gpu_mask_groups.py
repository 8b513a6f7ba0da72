"""Mask compaction where its launches change: masks that one launch counts for itself, groups of chunks,
more groups than are added up; offsets that begin between two 16-byte boundaries, any stride."""
import pytest
import torch

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 4097, 98303, 98304, 98305, 262144, 8388608, 8388609, 327680, 327681, 65536 * 17 + 4096, (1 << 26) + 5))
def test_positions_around_the_limits(n):
    import paper_1810_08723_amd as ocn
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    for density in (0.0, 0.03, 0.5, 1.0) if n < 1 << 20 else (0.5,):
        flags = torch.rand(n, generator=gen, device="cuda:0") < density
        want = torch.nonzero(flags).reshape(-1)
        m = ocn.Tensor(flags.data_ptr(), "bool", (n,), (1,), 0, 0, flags)
        for first, stride, capacity in ((0, 8, n), (1, -24, n), (1, 1, max(1, want.numel() - 2)), (0, 4, min(n, 7))):
            print("positions", n, density, first, stride, capacity, flush=True)
            out = torch.full((capacity + 2,), -9, dtype=torch.int64, device="cuda:0")
            count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
            ocn.mask_offsets(m, [stride], out[first:first + capacity], count)
            torch.cuda.synchronize()
            k = min(capacity, int(want.numel()))
            assert int(count.cpu()[0]) == int(want.numel())
            assert bool((out[first:first + k] == want[:k] * stride).all())
            assert bool((out[:first] == -9).all()) and bool((out[first + k:] == -9).all())


def test_positions_of_a_permuted_target():
    # two dims that do not merge: the general form of the writing kernel behind groups of chunks
    import paper_1810_08723_amd as ocn
    rows, cols = 1100, 517
    gen = torch.Generator(device="cuda:0").manual_seed(5)
    flags = torch.rand(rows, cols, generator=gen, device="cuda:0") < 0.4
    i = torch.nonzero(flags)
    want = i[:, 0] * 4 + i[:, 1] * 4 * rows
    out = torch.full((rows * cols,), -9, dtype=torch.int64, device="cuda:0")
    count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    ocn.mask_offsets(ocn.Tensor(flags.data_ptr(), "bool", (rows, cols), (cols, 1), 0, 0, flags), [4, 4 * rows], out, count)
    torch.cuda.synchronize()
    k = int(want.numel())
    assert int(count.cpu()[0]) == k and bool((out[:k] == want).all()) and bool((out[k:] == -9).all())
