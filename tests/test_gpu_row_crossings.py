"""Elementwise rows whose vectors go on into the next row, inputs that do not run along with the output: row
lengths around a vector and odd ones, inputs broadcast along either dim, reversed rows, rows that start
anywhere, several outer dims, byte order, outputs that start inside a vector."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

TYPES = ("bool", "int8", "int16", "half", "int32", "float", "double", "cfloat", "cdouble")


def _binary(dtype):
    return "lor" if dtype == "bool" else "add"


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("cols", (3, 4, 5, 8, 9, 15, 16, 17, 31, 41, 666, 1001))
def test_products_with_rows_and_columns(dtype, cols):
    rng = rng_for(28000 + cols)
    rows = 5000 // cols + 3
    a = random_view(rng, dtype, (rows, cols))
    row, column = random_view(rng, dtype, (1, cols)), random_view(rng, dtype, (rows, 1))
    wide = random_view(rng, dtype, (rows, cols + 3)).slice(1, 1, cols + 1, 1)
    out = View.empty(dtype, (rows, cols))
    for b in (row, column, wide, a.flip(0)):
        print("crossings", dtype, a.sizes, b.sizes, b.strides, flush=True)
        H.check_binary(_binary(dtype), a, b, out)
        H.check_binary(_binary(dtype), b, row, View.empty(dtype, tuple(np.broadcast_shapes(b.sizes, row.sizes))))
    flat = View.empty(dtype, (rows * cols + 1,))
    off = View(flat.storage, dtype, (rows, cols), out.strides, flat.strides[0])     # the output starts an element into a vector
    H.check_binary(_binary(dtype), wide, row, off)
    if dtype not in ("bool", "int8"):
        H.check_binary(_binary(dtype), wide.in_other_byte_order(), row.in_other_byte_order(), out)


@pytest.mark.parametrize("dtype", TYPES)
@pytest.mark.parametrize("cols", (2, 7, 13, 33, 250))
def test_copies_of_reversed_and_stepped_rows(dtype, cols):
    rng = rng_for(28200 + cols)
    x = random_view(rng, dtype, (7, 24, cols))
    for a in (x.flip(1), x.flip(0), x.slice(1, 0, 24, 2), x.permute(1, 0, 2)):
        print("crossings", dtype, a.sizes, a.strides, flush=True)
        H.check_unary("ident", a, View.empty(dtype, a.sizes))
