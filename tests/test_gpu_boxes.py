"""Boxes of any extents: permuted operands with short, odd and long axes, runs that go on along several
axes, boxes clipped by the end of the tensor, operands off by a few elements, inputs read in place,
broadcast, in the other byte order, and with rows an odd number of scalars apart."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

TYPES = [("add", "float", "float", "float"), ("mul", "cfloat", "cfloat", "cfloat"), ("absgt", "cfloat", "cfloat", "bool"),
         ("max", "uint8", "uint8", "uint8"), ("mul", "cdouble", "cdouble", "cdouble"), ("sub", "half", "float", "float"),
         (None, "double", None, "int16"), (None, "uint8", None, "float"), (None, "float", None, "uint8"), ("add", "half", "half", "half")]


def _stored(rng, dtype, shape, perm, shift):
    """A view of `shape` whose storage holds the dims in the order `perm`, `shift` elements in."""
    n = int(np.prod(shape))
    flat = random_view(rng, dtype, (n + 16,)) if rng is not None else View.empty(dtype, (n + 16,))
    es = flat.strides[0]
    strides, acc = [0] * len(shape), es
    for p in reversed(perm):
        strides[p] = acc
        acc *= shape[p]
    return View(flat.storage, dtype, tuple(shape), tuple(strides), flat.offset + shift * es)


@pytest.mark.parametrize("kind", range(len(TYPES)))
@pytest.mark.parametrize("shape", [(3, 40, 2, 17), (5, 25, 5, 38), (2, 3, 4, 5, 6), (97, 3, 33), (7, 66, 11, 13), (1300, 3, 5)])
def test_permuted_views(kind, shape):
    op, da, db, dout = TYPES[kind]
    rng = rng_for(23000 + 10 * kind + sum(shape))
    dims = list(range(len(shape)))
    orders = [(dims[1:] + dims[:1], dims[2:] + dims[:2]), (dims[::-1], dims), (dims[:-2] + [dims[-1], dims[-2]], dims[1:] + dims[:1])]
    for shift, (pa, pb) in enumerate(orders):
        print("boxes", TYPES[kind], shape, pa, pb, flush=True)
        a, out = _stored(rng, da, shape, pa, shift), _stored(None, dout, shape, dims, shift)
        if op is None:
            H.check_unary("ident", a, out)
        else:
            H.check_binary(op, a, _stored(rng, db, shape, pb, 3 * shift), out)


def test_broadcast_in_place_and_byte_order():
    rng = rng_for(23500)
    for shape in ((6, 35, 21), (40, 9, 70)):
        perm = (2, 0, 1)
        for dt in ("float", "half", "uint8", "double"):
            print("broadcast", dt, shape, flush=True)
            a = _stored(rng, dt, shape, perm, 1)
            for bs in ((1, 1, shape[2]), (shape[0], 1, 1), (1, shape[1], 1), (1, 1, 1)):
                H.check_binary("add", a, random_view(rng, dt, bs), View.empty(dt, shape))
                H.check_binary("sub", random_view(rng, dt, bs), a, View.empty(dt, shape))
            same = _stored(rng, dt, shape, (0, 1, 2), 0)
            H.check_binary("add", a, same, same)
        s = _stored(rng, "float", (shape[0], shape[2], shape[1]), (0, 1, 2), 0).in_other_byte_order().permute(0, 2, 1)
        H.check_binary("add", s, random_view(rng, "float", shape), View.empty("float", shape))


def test_many_boxes():
    # enough boxes that they are numbered in groups, with a remainder; runs longer than a box
    rng = rng_for(23600)
    for shape, perm in (((61, 45, 267), (2, 0, 1)), ((3, 5, 1021, 31), (3, 2, 0, 1)), ((9, 40001), (1, 0))):
        for dt in ("float", "cfloat", "uint8"):
            print("many boxes", dt, shape, flush=True)
            H.check_binary("add", _stored(rng, dt, shape, perm, 1), random_view(rng, dt, shape), View.empty(dt, shape))


@pytest.mark.parametrize("dt,sc", [("cfloat", 4), ("chalf", 2), ("cdouble", 8)])
def test_complex_rows_an_odd_number_of_scalars_apart(dt, sc):
    rng = rng_for(23700 + sc)
    for rows, cols in ((6, 40), (37, 70), (300, 5)):
        for apart, shift in ((1, 0), (3, 0), (2 * cols + 1, 1)):
            store = random_view(rng, dt, (rows * cols * 2 + rows * 2 + 8,), specials=False)
            a = View(store.storage, dt, (2, rows, cols), (0, apart * sc, 2 * sc), shift * sc)
            print("odd complex strides", dt, rows, cols, apart, shift, flush=True)
            H.check_binary("add", a, _stored(rng, dt, (2, rows, cols), (2, 0, 1), 0), View.empty(dt, (2, rows, cols)))
