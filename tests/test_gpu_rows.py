"""Rows of any length and alignment on the GPU: vectors that cross rows, partial vectors at both
ends, inputs off by a few elements, broadcast along either dim, reversed rows, outputs with gaps."""
from dataclasses import replace

import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

KINDS = [("mul", "int32", "float", "float"), ("add", "uint8", "uint8", "uint8"), ("gt", "double", "double", "bool"),
         ("mul", "cdouble", "cdouble", "cdouble"), ("sub", "half", "half", "half"),
         (None, "double", None, "int16"), (None, "uint8", None, "float"), (None, "half", None, "half")]


def _off_by(rng, dtype, shape, k):
    """A contiguous [rows, cols] view that starts k elements into its storage."""
    n = shape[0] * shape[1]
    flat = random_view(rng, dtype, (n + 24,)) if rng is not None else View.empty(dtype, (n + 24,))
    v = flat.slice(0, k, k + n, 1)
    return View(v.storage, dtype, shape, (shape[1] * v.strides[0], v.strides[0]), v.offset)


@pytest.mark.parametrize("kind", range(len(KINDS)))
@pytest.mark.parametrize("rows,cols", [(1, 1), (5, 3), (9, 16), (33, 17), (7, 255), (64, 257), (3, 4099)])
def test_ragged_rows(kind, rows, cols):
    op, da, db, dout = KINDS[kind]
    rng = rng_for(21000 + 100 * kind + rows)
    for k in (0, 1, 5):
        a = _off_by(rng, da, (rows, cols), k)
        out = _off_by(None, dout, (rows, cols), (3 * k) % 16)
        gaps = View.empty(dout, (rows, cols + 3)).slice(1, 1, cols + 1, 1)
        print("ragged rows", KINDS[kind], rows, cols, k, flush=True)
        for src in (a, a.flip(0)):
            if op is None:
                H.check_unary("ident", src, out)
                H.check_unary("ident", src, gaps)
            else:
                row = random_view(rng, db, (1, cols))
                col = random_view(rng, db, (rows, 1))
                H.check_binary(op, src, row.broadcast_to((rows, cols)), out)
                H.check_binary(op, col.broadcast_to((rows, cols)) if da == db else src, src if da == db else
                               col.broadcast_to((rows, cols)), out)
                H.check_binary(op, src, _off_by(rng, db, (rows, cols), (k + 2) % 7), gaps)
    if op is not None and da == dout:     # in place, with rows that end inside a vector
        a = _off_by(rng, da, (rows, cols), 1)
        H.check_binary(op, a, random_view(rng, db, (1, cols)).broadcast_to((rows, cols)), a)


@pytest.mark.parametrize("swap", (1, 2, 4, 7))
def test_ragged_rows_in_the_other_byte_order(swap):
    rng = rng_for(21900 + swap)
    a, b, out = _off_by(rng, "float", (19, 37), 1), random_view(rng, "float", (1, 37)), View.empty("float", (19, 37))
    a, b, out = (replace(v, byteswapped=True) if swap & bit else v for bit, v in ((1, a), (2, b), (4, out)))
    H.check_binary("add", a, b, out)


def test_three_outer_dims_and_long_rows():
    rng = rng_for(21990)
    a = random_view(rng, "float", (5, 7, 3, 1001)).flip(1).flip(2)
    H.check_unary("neg", a, View.empty("float", (5, 7, 3, 1001)))
    H.check_unary("ident", a, View.empty("half", (5, 7, 3, 1001)))
    b = random_view(rng, "float", (1, 7, 1, 1001))
    H.check_binary("mul", a, b, View.empty("float", (5, 7, 3, 1001)))
    H.check_binary("mul", b, a, View.empty("float", (5, 8, 3, 1003)).slice(1, 0, 7, 1).slice(3, 2, 1003, 1))


def test_rows_longer_than_two_to_the_31():
    # uint8 rows of 2^31 + 5 elements plus one element per row: every element is written and nothing
    # behind the output is.  Reference: the same sums on the device (wrapping, as the library's).
    import torch
    import paper_1810_08723_amd as ocn
    n = (1 << 31) + 5
    a = torch.randint(0, 256, (2, n), dtype=torch.uint8, device="cuda:0")
    b = torch.tensor([[7], [201]], dtype=torch.uint8, device="cuda:0")
    out = torch.full((2 * n + 64,), 0x5A, dtype=torch.uint8, device="cuda:0")
    print("rows of", n, flush=True)
    ocn.binary("add", ocn.Tensor(a.data_ptr(), "uint8", (2, n), (n, 1), 0, 0, a),
               ocn.Tensor(b.data_ptr(), "uint8", (2, 1), (1, 1), 0, 0, b),
               ocn.Tensor(out.data_ptr(), "uint8", (2, n), (n, 1), 0, 0, out))
    torch.cuda.synchronize()
    a.add_(b)
    for row in range(2):
        for lo in range(0, n, 1 << 28):
            hi = min(n, lo + (1 << 28))
            assert torch.equal(out[row * n + lo:row * n + hi], a[row, lo:hi]), (row, lo)
    assert bool((out[2 * n:] == 0x5A).all())
