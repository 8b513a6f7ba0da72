"""Masks around the sizes where a workgroup takes a quarter of a chunk: edges of quarters and chunks, both ways to
count what lies before, any mask byte that is not zero, too small a capacity, and the first size beyond."""
import numpy as np
import pytest

from workloads.values import rng_for

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("n", (1, 3, 5, 1023, 1024, 1025, 4095, 4097, 5121, 8191, 36865, 98303, 98304, 98305, 102399,
                               (1 << 20) - 1, 1 << 20, (1 << 20) + 1))
@pytest.mark.parametrize("density", (0.02, 0.6, 1.0))
def test_quarters_of_chunks(n, density):
    import torch
    import paper_1810_08723_amd as ocn
    rng = rng_for(26700 + n)
    flags = np.where(rng.random(n) < density, rng.choice(np.array([1, 2, 0x7f, 0x80, 0xff], np.uint8), n), 0).astype(np.uint8)
    want = np.flatnonzero(flags).astype(np.int64) * -12
    store = np.full(n + 16, 0xff, np.uint8)            # bytes behind the mask are not part of it
    store[:n] = flags
    mask = torch.from_numpy(store).to("cuda:0")
    m = ocn.Tensor(mask.data_ptr(), "bool", (n,), (1,), 0, 0, mask)
    for capacity in sorted({n, len(want), max(0, len(want) - 1), len(want) // 2}):
        for shift in (0, 1):                           # offsets that start on 16 bytes and between
            out = torch.full((n + 2,), -9, dtype=torch.int64, device="cuda:0")
            count = torch.full((1,), 77, dtype=torch.int64, device="cuda:0")
            print("quarters", n, density, capacity, shift, flush=True)
            ocn.mask_offsets(m, [-12], out[shift:shift + capacity], count)
            got = out.cpu().numpy()
            k = min(capacity, len(want))
            assert int(count.cpu()[0]) == len(want)
            assert np.array_equal(got[shift:shift + k], want[:k]) and (np.delete(got, np.arange(shift, shift + k)) == -9).all()
