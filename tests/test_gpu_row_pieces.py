"""Inputs whose vectors go on into the next row, on both sides of the rule that takes them in two whole pieces: rows
around a vector, long rows of bytes in small and large outputs, flat calls of odd lengths, one input and two."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

NUMPY = {"int8": np.int8, "uint8": np.uint8, "int16": np.int16, "float": np.float32}


@pytest.mark.parametrize("dtype,rows,cols", [(d, 4001, w) for d in NUMPY for w in (3, 4, 7, 8, 9, 15, 16, 17, 33)] +
                         [("int8", 700, 1023), ("int8", 8200, 1023), ("int8", 8195, 1024), ("int8", 8180, 1025), ("uint8", 1001, 1025), ("uint8", 3001, 3001), ("int16", 3001, 3001)])
@pytest.mark.parametrize("how", ("row", "column", "reversed", "wide"))
def test_both_sides_of_the_rule(dtype, rows, cols, how):
    rng = rng_for(34000 + rows + cols)
    a = random_view(rng, dtype, (rows, cols), specials=False)
    b = random_view(rng, dtype, {"row": (1, cols), "column": (rows, 1), "reversed": (rows, cols), "wide": (rows, cols + 3)}[how], specials=False)
    if how == "reversed":
        b = b.flip(0)
    elif how == "wide":
        b = b.slice(1, 1, cols + 1)
    for x, y in ((a, b), (b, a)):
        out = View.empty(dtype, (rows, cols))
        print("pieces", dtype, rows, cols, how, flush=True)
        H.check_binary("add", x, y, out)
    out = View.empty(dtype, b.sizes)
    H.check_unary("neg", b, out)


@pytest.mark.parametrize("dtype", ("int8", "half", "float", "double", "cfloat"))
@pytest.mark.parametrize("n", (1, 15, 16, 17, 4097, 100003))
def test_flat_calls_of_any_length(dtype, n):
    rng = rng_for(34200 + n)
    a, b = (random_view(rng, dtype, (n,), specials=False) for _ in range(2))
    print("flat", dtype, n, flush=True)
    H.check_binary("add", a, b, View.empty(dtype, (n,)))
    H.check_unary("neg", a, View.empty(dtype, (n,)))
