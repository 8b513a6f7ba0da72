"""Column reductions whose lanes are numbered through whole rows of equal column blocks: shapes that take
that form, remainders of columns and rows, several kept dims, rows that start anywhere, byte order."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

# (the last nine take the form for the types in FLAT; the others for some types, and the forms beside it)
SHAPES = [(100, 500, 260), (3, 40, 300, 260), (64, 129, 516), (100, 131, 400), (30, 128, 1001),
          (48, 1000, 777), (3, 257, 777), (2, 200, 1300), (5, 200, 1040), (3, 515, 1040),
          (19, 49, 3546), (179, 55, 601), (69, 76, 1699), (1, 300, 33003)]
VECTOR = {"int32": 4, "int64": 2, "int16": 8, "float": 4, "double": 2, "half": 8, "cfloat": 2}
FLAT = {(48, 1000, 777): (2, 4, 8), (3, 257, 777): (2, 4, 8), (2, 200, 1300): (2, 4, 8), (5, 200, 1040): (2, 4), (3, 515, 1040): (8,),
        (19, 49, 3546): (2,), (179, 55, 601): (4,), (69, 76, 1699): (8,), (1, 300, 33003): (2, 4, 8)}


def _in_equal_blocks(op, a, axis, out, vec):
    """Are the columns cut into blocks of another number of lanes than a power of two?"""
    import paper_1810_08723_amd as ocn
    p = ocn.plan_reduce(op, ocn.Tensor(0x1000000000, a.dtype, a.sizes, a.strides, a.offset, 0, byteswapped=getattr(a, "byteswapped", False)), [axis],
                        ocn.Tensor(0x2000000000, out.dtype, out.sizes, out.strides, out.offset, 0))
    lanes, others = -(-a.sizes[-1] // vec), int(np.prod(out.sizes[:-1]))
    return p["kernel"] == "red_cols" and p["vec"] == vec and p["split"] == 1 and all(p["grid"] != -(-lanes // c) * others for c in (1, 2, 4, 8, 16, 32, 64))


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("dtype", ("int32", "int64", "int16", "float", "double", "half", "cfloat"))
def test_equal_column_blocks(shape, dtype):
    rng = rng_for(25000 + sum(shape))
    axis = len(shape) - 2
    x = random_view(rng, dtype, shape, specials=False)
    variants = [x, x.slice(len(shape) - 1, 1, shape[-1], 1)]
    if dtype != "half":
        variants.append(random_view(rng, dtype, shape, specials=False).in_other_byte_order())
    exact = dtype.startswith("int")
    for a in variants:
        kept = [n for d, n in enumerate(a.sizes) if d != axis]
        for op in ("sum", "max") if dtype != "cfloat" else ("sum",):
            out = View.empty(("int64" if exact else dtype) if op == "sum" else dtype, kept)
            assert VECTOR[dtype] not in FLAT.get(shape, ()) or _in_equal_blocks(op, a, axis, out, VECTOR[dtype]), (op, dtype, a.sizes)
            print("flat columns", op, dtype, a.sizes, a.strides, flush=True)
            got, want = H.run_reduce(op, a, (axis,), out)
            if exact or op == "max":
                assert H.storages_equal(out.dtype, got, want), (op, dtype, shape, H.first_mismatch(out.dtype, got, want))
            else:   # 64-bit accumulators, one rounding to the output: 1 unit of it and the order of the sum
                comp = {"float": np.float32, "cfloat": np.float32, "double": np.float64, "half": np.float16}[dtype]
                g, w = got.view(comp).astype(np.float64), want.view(comp).astype(np.float64)
                native = np.abs(a.to_numpy())
                mag = native.astype(np.float64).sum(axis=axis).reshape(-1)
                if dtype == "cfloat":
                    mag = np.repeat(mag, 2)
                rel = {"float": 1e-6, "cfloat": 1e-6, "double": 1e-13, "half": 1e-3}[dtype]
                fin = np.isfinite(w)
                assert np.array_equal(np.isfinite(g), fin) and np.all(np.abs(g[fin] - w[fin]) <= rel * mag[fin] + 1e-300)
