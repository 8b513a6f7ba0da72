"""The generic-dtype kernel on rows of any length and alignment: groups of four that end with the
row, broadcast inputs, in place, the other byte order."""
from dataclasses import replace

import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

KINDS = [("mul", "bool", "float", "float"), ("add", "int16", "float", "double"), ("lt", "int32", "int64", "bool"),
         ("sub", "int8", "uint16", "half"), ("mul", "half", "cfloat", "cdouble"), ("band", "uint8", "int32", "int64")]


def _off_by(rng, dtype, shape, k):
    n = shape[0] * shape[1]
    flat = random_view(rng, dtype, (n + 8,)) if rng is not None else View.empty(dtype, (n + 8,))
    es = flat.strides[0]
    return View(flat.storage, dtype, shape, (shape[1] * es, es), flat.offset + k * es)


@pytest.mark.parametrize("kind", range(len(KINDS)))
@pytest.mark.parametrize("cols", (1, 3, 4, 5, 6, 7, 63, 257))
def test_generic_rows(kind, cols):
    import paper_1810_08723_amd as ocn
    op, da, db, dout = KINDS[kind]
    rng = rng_for(25000 + 10 * kind + cols)
    rows = 13
    for k in (0, 1):
        a, b = _off_by(rng, da, (rows, cols), k), _off_by(rng, db, (rows, cols), 3 * k)
        out = _off_by(None, dout, (rows, cols), k)
        if cols > 1:
            plan = ocn.plan_binary(op, *(ocn.Tensor(1 << (40 + i), v.dtype, v.sizes, v.strides, v.offset, 0)
                                         for i, v in enumerate((a, b, out))))
            assert not plan["specialised"]
        print("generic rows", KINDS[kind], cols, k, flush=True)
        H.check_binary(op, a, b, out)
        H.check_binary(op, a, random_view(rng, db, (1, cols)), out)
        H.check_binary(op, random_view(rng, da, (rows, 1)), b, View.empty(dout, (rows, cols + 2)).slice(1, 1, cols + 1, 1))
        H.check_binary(op, a.flip(0), replace(b, byteswapped=True), out)


@pytest.mark.parametrize("cols", (4, 5, 7, 130))
def test_in_place_on_generic_types(cols):
    rng = rng_for(25500 + cols)
    a = _off_by(rng, "float", (9, cols), 1)
    H.check_binary("mul", a, random_view(rng, "int16", (9, cols)), a)           # float *= int16
    b = _off_by(rng, "double", (9, cols), 1)
    H.check_binary("sub", random_view(rng, "uint16", (1, cols)), b, b)
