"""Index arrays around the two sizes between which one workgroup counts the invalid indices and the others bind:
both parities, both tensors, their alignment, offsets in place of the indices, a cap on workgroups, replays."""
import numpy as np
import pytest

from workloads.values import rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dim,stride", ((997, 24), (1, -8), (0, 8), (1 << 40, 1 << 20)))
@pytest.mark.parametrize("n", (4095, 4096, 4097, 4098, 6144, 6145, 6146, 16382, 16383, 16384, 16385))
def test_counted_beside_the_offsets(n, dim, stride):
    import torch
    import paper_1810_08723_amd as ocn
    from oracle import indexing as OI
    rng = rng_for(26300 + n)
    idx = rng.integers(-dim - dim // 9 - 1, dim + dim // 9 + 2, size=n).astype(np.int64)
    idx[[0, -1]] = dim, -dim - 1                       # out of range, the last of an odd number too
    want, bad = OI.index_offsets(idx, dim, stride)
    for si, so, cap in ((0, 0, None), (1, 0, None), (0, 1, None), (0, 0, 2)):
        src = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
        src[si:si + n] = torch.from_numpy(idx).to("cuda:0")
        out = torch.full((n + 3,), -5, dtype=torch.int64, device="cuda:0")
        count = torch.full((1,), 77, dtype=torch.int64, device="cuda:0")
        print("counted", n, dim, si, so, cap, flush=True)
        if cap:
            ocn.binding.set_max_launch_blocks(cap)
        try:
            ocn.index_offsets(ocn.Tensor(src.data_ptr(), "int64", (n,), (8,), 8 * si, 0, src), dim, stride,
                              ocn.Tensor(out.data_ptr(), "int64", (n,), (8,), 8 * so, 0, out), count)
        finally:
            if cap:
                ocn.binding.set_max_launch_blocks(0)
        got = out.cpu().numpy()
        assert np.array_equal(got[so:so + n], want) and int(count.cpu()[0]) == bad
        assert (np.delete(got, np.arange(so, so + n)) == -5).all()
    t = torch.from_numpy(idx).to("cuda:0")             # the offsets replace the indices
    count = torch.full((1,), 77, dtype=torch.int64, device="cuda:0")
    v = ocn.Tensor(t.data_ptr(), "int64", (n,), (8,), 0, 0, t)
    ocn.index_offsets(v, dim, stride, v, count)
    assert np.array_equal(t.cpu().numpy(), want) and int(count.cpu()[0]) == bad


def test_counted_in_a_captured_graph():
    import torch
    import paper_1810_08723_amd as ocn
    from oracle import indexing as OI
    n, dim = 9001, 500
    src = torch.zeros(n, dtype=torch.int64, device="cuda:0")
    out = torch.zeros(n, dtype=torch.int64, device="cuda:0")
    count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
    a = ocn.Tensor(src.data_ptr(), "int64", (n,), (8,), 0, 0, src)
    b = ocn.Tensor(out.data_ptr(), "int64", (n,), (8,), 0, 0, out)
    ocn.index_offsets(a, dim, 8, b, count)
    torch.cuda.synchronize()
    graph = torch.cuda.CUDAGraph()
    with torch.cuda.graph(graph):
        ocn.index_offsets(a, dim, 8, b, count)
    for replay in range(4):
        idx = rng_for(26500 + replay).integers(-2 * dim, 2 * dim, size=n).astype(np.int64)
        src.copy_(torch.from_numpy(idx).to("cuda:0"))
        out.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        want, bad = OI.index_offsets(idx, dim, 8)
        assert np.array_equal(out.cpu().numpy(), want) and int(count.cpu()[0]) == bad
