"""Index binding, mask compaction, gather and scatter around the sizes where their launches change:
index arrays of one workgroup and more, masks counted directly, by chunk sums and by a scan, rows
of every length from one element, whole and partial pieces, any alignment, both byte orders."""
import numpy as np
import pytest

from workloads.values import rng_for

pytestmark = pytest.mark.gpu

NP = {"uint8": np.uint8, "half": np.float16, "float": np.float32, "double": np.float64, "cdouble": np.complex128}


@pytest.mark.parametrize("n", (1, 7, 1023, 16384, 16385, 70001))
def test_index_binding_around_one_workgroup(n):
    import torch
    import paper_1810_08723_amd as ocn
    from oracle import indexing as OI
    rng = rng_for(24000 + n)
    dim = 1000
    idx = rng.integers(-dim - 40, dim + 40, size=n).astype(np.int64)
    for shift in (0, 1):                       # an index array that is 16-byte aligned and one that is not
        src = torch.zeros(n + 1, dtype=torch.int64, device="cuda:0")
        src[shift:shift + n] = torch.from_numpy(idx).to("cuda:0")
        out = torch.full((n + 2,), -5, dtype=torch.int64, device="cuda:0")
        bad = torch.full((1,), 77, dtype=torch.int64, device="cuda:0")
        ti = ocn.Tensor(src.data_ptr(), "int64", (n,), (8,), 8 * shift, 0, src)
        to = ocn.Tensor(out.data_ptr(), "int64", (n,), (8,), 8, 0, out)
        ocn.index_offsets(ti, dim, 24, to, bad)
        want, want_bad = OI.index_offsets(idx, dim, 24)
        got = out.cpu().numpy()
        assert np.array_equal(got[1:n + 1], want) and int(bad.cpu()[0]) == want_bad
        assert got[0] == -5 and got[n + 1] == -5


@pytest.mark.parametrize("n", (1, 15, 4096, 4097, 16384, 16385, 65536, 65537, 81920, 300001, (1 << 25) + 4097))
@pytest.mark.parametrize("density", (0.0, 0.03, 0.5, 1.0))
def test_mask_compaction_sizes(n, density):
    import torch
    import paper_1810_08723_amd as ocn
    if n > 1 << 25 and density != 0.5:
        pytest.skip("the largest size once")
    gen = torch.Generator(device="cuda:0").manual_seed(n)
    flags = torch.rand(n + 3, generator=gen, device="cuda:0") < density
    for shift in (0, 3) if n < 1 << 20 else (0,):          # a contiguous, aligned mask and one that is not aligned
        mask = flags[shift:shift + n]
        want = torch.nonzero(mask).reshape(-1) * 4
        m = ocn.Tensor(flags.data_ptr(), "bool", (n,), (1,), shift, 0, flags)
        for capacity in {n, max(1, int(want.numel()) - 1)}:
            out = torch.full((capacity + 1,), -9, dtype=torch.int64, device="cuda:0")
            count = torch.zeros(1, dtype=torch.int64, device="cuda:0")
            print("mask", n, density, shift, capacity, flush=True)
            ocn.mask_offsets(m, [4], out[:capacity], count)
            torch.cuda.synchronize()
            k = min(capacity, int(want.numel()))
            assert int(count.cpu()[0]) == int(want.numel())
            assert bool((out[:k] == want[:k]).all()) and bool((out[k:] == -9).all())


@pytest.mark.parametrize("dtype", ("uint8", "half", "float", "double", "cdouble"))
@pytest.mark.parametrize("width", (1, 2, 3, 5, 7, 8, 17, 33, 75, 1025))
def test_rows_of_every_length(dtype, width):
    import torch
    import paper_1810_08723_amd as ocn
    rng = rng_for(24500 + width)
    es = np.dtype(NP[dtype]).itemsize
    table, n = 137, 90 if width > 100 else 3000
    raw = rng.integers(0, 256, size=table * width * es, dtype=np.uint8)
    rows = raw.reshape(table, width * es)
    pick = rng.integers(0, table, size=n)
    lo, hi = width * es, (table - 2) * width * es          # the first and the last row are out of range: skipped
    for shift in (0, es):
        for swap in (False, True) if es > 1 and dtype != "cdouble" else (False,):
            src = torch.zeros(raw.size + shift, dtype=torch.uint8, device="cuda:0")
            src[shift:] = torch.from_numpy(raw).to("cuda:0")
            offs = torch.from_numpy(pick.astype(np.int64) * width * es).to("cuda:0")
            out = torch.full((n * width * es + 2 * es,), 0xA5, dtype=torch.uint8, device="cuda:0")
            ti = ocn.Tensor(src.data_ptr(), dtype, (width,), (es,), shift, 0, src)
            to = ocn.Tensor(out.data_ptr(), dtype, (n, width), (width * es, es), es, 0, out, swap)
            print("rows", dtype, width, shift, swap, flush=True)
            ocn.gather(ti, offs, lo, hi, to)
            want = rows[pick].copy()
            if swap:
                want = want.reshape(n, width, es)[:, :, ::-1].reshape(n, width * es)
            want[(pick == 0) | (pick == table - 1)] = 0xA5
            got = out.cpu().numpy()
            assert np.array_equal(got[es:-es].reshape(n, -1), want)
            assert (got[:es] == 0xA5).all() and (got[-es:] == 0xA5).all()
            # and back: every row of the table at most once
            perm = rng.permutation(table)[:min(n, table)]
            vals = torch.from_numpy(rng.integers(0, 256, size=len(perm) * width * es, dtype=np.uint8)).to("cuda:0")
            dst = torch.full((raw.size + 2 * es,), 0x5A, dtype=torch.uint8, device="cuda:0")
            tv = ocn.Tensor(vals.data_ptr(), dtype, (len(perm), width), (width * es, es), 0, 0, vals, swap)
            td = ocn.Tensor(dst.data_ptr(), dtype, (width,), (es,), es, 0, dst)
            ocn.scatter(tv, torch.from_numpy(perm.astype(np.int64) * width * es).to("cuda:0"), lo, hi, td)
            want = np.full((table, width * es), 0x5A, dtype=np.uint8)
            v = vals.cpu().numpy().reshape(len(perm), width, es)
            want[perm] = (v[:, :, ::-1] if swap else v).reshape(len(perm), -1)
            want[[0, table - 1]] = 0x5A
            got = dst.cpu().numpy()
            assert np.array_equal(got[es:-es].reshape(table, -1), want)
            assert (got[:es] == 0x5A).all() and (got[-es:] == 0x5A).all()


@pytest.mark.parametrize("dtype,width,n", [("float", 7, 131077), ("uint8", 5, 131079), ("uint8", 3, 140001), ("half", 33, 52433),
                                           ("double", 3, 131083), ("float", 75, 13801), ("uint8", 4099, 1021)])
def test_four_pieces_per_lane(dtype, width, n):
    """Enough pieces that a lane takes four (262144 and more): rows that are no multiple of a piece, the
    base off by one element, the other byte order, offsets out of range, a ragged last workgroup."""
    import torch
    import paper_1810_08723_amd as ocn
    rng = rng_for(24900 + width)
    es = np.dtype(NP[dtype]).itemsize
    table = n + 11
    row = width * es
    raw = rng.integers(0, 256, size=(table, row), dtype=np.uint8)
    pick = rng.permutation(table)[:n]
    lo, hi = 2 * row, (table - 3) * row
    skipped = (pick < 2) | (pick > table - 3)
    offs = torch.from_numpy(pick.astype(np.int64) * row).to("cuda:0")
    for swap in (False, True) if es > 1 else (False,):
        turned = lambda x: x.reshape(len(x), width, es)[:, :, ::-1].reshape(len(x), row) if swap else x
        src = torch.zeros(raw.size + es, dtype=torch.uint8, device="cuda:0")
        src[es:] = torch.from_numpy(raw.reshape(-1)).to("cuda:0")
        out = torch.full((n * row + 2 * es,), 0xA5, dtype=torch.uint8, device="cuda:0")
        print("four pieces", dtype, width, n, swap, flush=True)
        ocn.gather(ocn.Tensor(src.data_ptr(), dtype, (width,), (es,), es, 0, src), offs, lo, hi,
                   ocn.Tensor(out.data_ptr(), dtype, (n, width), (row, es), es, 0, out, swap))
        want = turned(raw[pick]).copy()
        want[skipped] = 0xA5
        got = out.cpu().numpy()
        assert np.array_equal(got[es:-es].reshape(n, row), want)
        assert (got[:es] == 0xA5).all() and (got[-es:] == 0xA5).all()
        vals = rng.integers(0, 256, size=(n, row), dtype=np.uint8)
        tv = torch.from_numpy(vals).to("cuda:0")
        dst = torch.full((table * row + 2 * es,), 0x5A, dtype=torch.uint8, device="cuda:0")
        ocn.scatter(ocn.Tensor(tv.data_ptr(), dtype, (n, width), (row, es), 0, 0, tv, swap), offs, lo, hi,
                    ocn.Tensor(dst.data_ptr(), dtype, (width,), (es,), es, 0, dst))
        want = np.full((table, row), 0x5A, dtype=np.uint8)
        want[pick[~skipped]] = turned(vals)[~skipped]
        got = dst.cpu().numpy()
        assert np.array_equal(got[es:-es].reshape(table, row), want)
        assert (got[:es] == 0x5A).all() and (got[-es:] == 0x5A).all()
