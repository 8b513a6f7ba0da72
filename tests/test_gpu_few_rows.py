"""Column reductions over a few rows, many times over: a lane per vector of columns.  Numbers of rows
around the loads in flight and the limit, columns below, at and above a vector, kept dims that do not
merge, rows that start anywhere, byte order."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ("int32", "int8", "int16", "double", "float", "half", "cfloat"))
@pytest.mark.parametrize("rows,cols", [(1, 4), (3, 2), (4, 15), (5, 33), (31, 8), (32, 9), (33, 7)])
def test_few_rows(dtype, rows, cols):
    rng = rng_for(26000 + 100 * rows + cols)
    n = 33000 // cols + 300
    x = random_view(rng, dtype, (n, rows, cols), specials=False)
    variants = [x, x.slice(2, 1, cols, 1)] + ([x.in_other_byte_order()] if dtype not in ("int8", "half") else [])
    y = random_view(rng, dtype, (20, rows, n // 20 + 1, cols), specials=False)     # two kept dims around the rows
    for a, axis in [(v, 1) for v in variants] + [(y, 1)]:
        kept = [s for d, s in enumerate(a.sizes) if d != axis]
        for op in ("max",) if dtype != "cfloat" and dtype not in ("int8", "int16", "int32") else ("sum",) if dtype == "cfloat" else ("sum", "max"):
            out = View.empty("int64" if op == "sum" and dtype != "cfloat" else dtype, kept)
            print("few rows", op, dtype, a.sizes, a.strides, flush=True)
            got, want = H.run_reduce(op, a, (axis,), out)
            if dtype == "cfloat":   # sums in 64 bits, rounded once
                g, w = got.view(np.float32).astype(np.float64), want.view(np.float32).astype(np.float64)
                fin = np.isfinite(w)
                assert np.array_equal(np.isfinite(g), fin)
                assert np.all(np.abs(g[fin] - w[fin]) <= 1.2e-7 * np.abs(w[fin]) + 1e-6 * rows * np.abs(w[fin]).max())
            else:
                assert H.storages_equal(out.dtype, got, want), (op, dtype, rows, cols, H.first_mismatch(out.dtype, got, want))
