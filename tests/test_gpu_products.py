"""Products of a matrix and a vector, and short inner products, at the sizes where their kernels change:
trips that end with fewer vectors than a lane takes, one workgroup for a whole output, columns with
either input broadcast along them."""
import numpy as np
import pytest

import gpu_harness as H
from test_gpu_fused import _check
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ("int32", "float", "double"))
@pytest.mark.parametrize("n", (256, 257, 260, 764, 1000, 1024, 1027, 2052))
def test_rows_of_odd_numbers_of_vectors(dtype, n):
    rng = rng_for(24000 + n)
    for rows in (1, 5, 130):
        a = random_view(rng, dtype, (rows, n), specials=False)
        _check("mul", "sum", a, random_view(rng, dtype, (1, n), specials=False), (1,), dtype)
        _check("lt", "sum", a, random_view(rng, dtype, (rows, n), specials=False), (1,), "bool", "int64")


@pytest.mark.parametrize("n", (8192, 16384, 16388, 32767, 32768, 32772, 65536, 65544, 131076))
def test_one_workgroup_per_output(n):
    rng = rng_for(24200 + n % 1000)
    for dtype, rows in (("int64", 1), ("float", 3), ("half", 2)):
        a = random_view(rng, dtype, (rows, n), specials=False)
        _check("mul", "sum", a, a.fresh_copy(), (1,), dtype)
    for dtype in ("int32", "uint8", "half"):
        x = random_view(rng, dtype, (3, n))
        for op in ("sum", "max") if dtype != "half" else ("max",):
            out = View.empty("int64" if op == "sum" else dtype, (3,))
            print("one workgroup", op, dtype, n, flush=True)
            got, want = H.run_reduce(op, x, (1,), out)
            assert H.storages_equal(out.dtype, got, want), (op, dtype, n, H.first_mismatch(out.dtype, got, want))


@pytest.mark.parametrize("dtype", ("int32", "float", "double", "cfloat"))
@pytest.mark.parametrize("shape", [(1, 8), (67, 33), (1712, 22), (500, 4), (130, 260), (40, 1000)])
def test_columns_with_a_broadcast_input(dtype, shape):
    rng = rng_for(24500 + sum(shape))
    v = random_view(rng, dtype, shape, specials=False)
    column = random_view(rng, dtype, (shape[0], 1), specials=False)
    _check("mul", "sum", v, column, (0,), dtype)
    _check("sub", "sum", column, v, (0,), dtype)
    _check("add", "sum", v, random_view(rng, dtype, (1, shape[1]), specials=False), (0,), dtype)
