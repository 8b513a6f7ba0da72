"""Column reductions over a few rows, many times over: a lane per vector of columns.  Numbers of rows
around the loads in flight and the limit, one column per lane and vectors of them, kept dims that do not
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


VECTOR = {"int32": 4, "int64": 2, "int16": 8, "float": 4, "double": 2, "half": 8, "cfloat": 2}


def _takes_lanes(op, a, axis, out, lanes_of):
    """Does the plan give every vector of columns a lane of its own (and how long are the vectors)?"""
    import paper_1810_08723_amd as ocn
    fake = [ocn.Tensor(base, v.dtype, v.sizes, v.strides, v.offset, 0, byteswapped=swapped) for base, v, swapped in
            ((0x1000000000, a, getattr(a, "byteswapped", False)), (0x2000000000, out, False))]
    p = ocn.plan_reduce(op, fake[0], [axis], fake[1])
    return p["kernel"] == "red_cols" and p["grid"] == -(-lanes_of(p["vec"]) // 256), p["vec"]


@pytest.mark.parametrize("dtype", sorted(VECTOR))
@pytest.mark.parametrize("rows,vectors,more", [(3, 1, 0), (4, 2, -1), (5, 3, 1), (32, 1, 0), (8, 40, 1), (31, 5, 2)])
def test_few_rows_in_vectors(dtype, rows, vectors, more):
    """As above with enough lanes for whole vectors: a last vector moved back over its neighbour, rows that
    start off their vectors, byte order, two kept dims beside the columns that do not merge."""
    rng = rng_for(26500 + 100 * rows + vectors)
    vec = VECTOR[dtype]
    cols = vectors * vec + more
    n = -(-32768 // -(-cols // vec)) + 1
    wide = 3 * n // (2 if vec == 8 and vectors >= 40 else 3)
    x = random_view(rng, dtype, (wide, rows, cols), specials=False)
    odd = random_view(rng, dtype, (wide, rows, cols + 1), specials=False).slice(2, 1, cols + 1, 1)
    y = random_view(rng, dtype, (11, rows, wide // 11 + 1, cols + 1), specials=False).slice(3, 0, cols, 1)
    variants = [x, odd, y] + ([x.in_other_byte_order(), odd.in_other_byte_order()] if dtype != "half" else [])
    for a in variants:
        kept = [s for d, s in enumerate(a.sizes) if d != 1]
        op = "max" if dtype in ("float", "double", "half") else "sum"
        out = View.empty("int64" if op == "sum" and dtype != "cfloat" else dtype, kept)
        others = int(np.prod(kept[:-1]))
        lanes, width = _takes_lanes(op, a, 1, out, lambda v: others * -(-cols // v))
        # (columns of 16 bits that start off their vectors are taken one by one unless rows are long)
        assert lanes and width in ((vec, 1) if vec == 8 else (vec,)), (dtype, a.sizes, a.strides, width)
        print("few rows in vectors", op, dtype, a.sizes, a.strides, width, flush=True)
        got, want = H.run_reduce(op, a, (1,), out)
        if dtype == "cfloat":   # sums in 64 bits, rounded once
            g, w = got.view(np.float32).astype(np.float64), want.view(np.float32).astype(np.float64)
            fin = np.isfinite(w)
            assert np.array_equal(np.isfinite(g), fin)
            assert np.all(np.abs(g[fin] - w[fin]) <= 1.2e-7 * np.abs(w[fin]) + 1e-6 * rows * np.abs(w[fin]).max())
        else:
            assert H.storages_equal(out.dtype, got, want), (op, dtype, a.sizes, H.first_mismatch(out.dtype, got, want))
