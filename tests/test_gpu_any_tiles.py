"""Tiles that the end of the tensor clips, and operands that are aligned to their elements only:
transposes and permutations with extents around the tile's, short axes, steps, operands off by a
few elements, in the forms with one and with two staged inputs."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

TYPES = [("add", "float", "float", "float"), ("mul", "cfloat", "cfloat", "cfloat"), ("absgt", "cfloat", "cfloat", "bool"),
         ("max", "uint8", "uint8", "uint8"), ("mul", "cdouble", "cdouble", "cdouble"), ("sub", "half", "float", "float"),
         (None, "double", None, "int16"), (None, "uint8", None, "float"), (None, "float", None, "uint8")]


def _stored(rng, dtype, shape, perm, shift):
    """A view of `shape` whose storage holds the dims in the order `perm`, `shift` elements in."""
    phys = [shape[p] for p in perm]
    n = int(np.prod(phys))
    flat = random_view(rng, dtype, (n + 16,)) if rng is not None else View.empty(dtype, (n + 16,))
    es = flat.strides[0]
    strides, acc = [0] * len(shape), es
    for p in reversed(perm):
        strides[p] = acc
        acc *= shape[p]
    return View(flat.storage, dtype, tuple(shape), tuple(strides), flat.offset + shift * es)


@pytest.mark.parametrize("kind", range(len(TYPES)))
@pytest.mark.parametrize("shape", [(3, 2), (31, 33), (64, 65), (127, 5), (2, 300), (333, 129)])
def test_clipped_transposes(kind, shape):
    op, da, db, dout = TYPES[kind]
    rng = rng_for(22000 + 10 * kind + shape[0])
    for shift in (0, 3):
        print("clipped transpose", TYPES[kind], shape, shift, flush=True)
        a, out = _stored(rng, da, shape, (1, 0), shift), _stored(None, dout, shape, (0, 1), shift)
        if op is None:
            H.check_unary("ident", a, out)
        else:
            H.check_binary(op, a, _stored(rng, db, shape, (0, 1), shift), out)
            H.check_binary(op, a, _stored(rng, db, shape, (1, 0), 1), out)
            if da == dout:
                same = _stored(rng, dout, shape, (0, 1), shift)
                H.check_binary(op, a, same, same)             # in place, the other operand staged


@pytest.mark.parametrize("kind", (0, 1, 2, 3, 5))
@pytest.mark.parametrize("shape", [(5, 7, 9), (2, 19, 37), (17, 3, 66), (6, 11, 4, 9), (3, 5, 2, 7, 13)])
def test_three_different_fastest_axes(kind, shape):
    op, da, db, dout = TYPES[kind]
    rng = rng_for(22500 + 10 * kind + len(shape) + shape[0])
    dims = list(range(len(shape)))
    for shift in (0, 1):
        a = _stored(rng, da, shape, dims[1:] + dims[:1], shift)
        b = _stored(rng, db, shape, dims[2:] + dims[:2], shift)
        print("three axes", TYPES[kind], shape, shift, flush=True)
        H.check_binary(op, a, b, _stored(None, dout, shape, dims, shift))
        H.check_binary(op, a, b, _stored(None, dout, shape, dims[::-1], 2))


def test_steps_gaps_and_byte_order():
    rng = rng_for(22900)
    a = random_view(rng, "float", (90, 70)).permute(1, 0).slice(0, 0, 69, 2)      # strided along its own fastest axis
    H.check_unary("neg", a, View.empty("float", a.sizes))
    H.check_binary("add", a, random_view(rng, "float", a.sizes), View.empty("float", (35, 97)).slice(1, 3, 93, 1))
    s = random_view(rng, "float", (53, 41)).in_other_byte_order().permute(1, 0)
    H.check_binary("add", s, random_view(rng, "float", (41, 53)), View.empty("float", (41, 53)))
    big = random_view(rng, "float", (700, 1301))                                   # more tiles than the small-launch rules take
    H.check_binary("add", big.permute(1, 0), random_view(rng, "float", (1301, 700)), View.empty("float", (1301, 700)))


def test_vectors_at_the_end_of_an_operand():
    # an operand that ends with its storage, of just one vector and of one element less
    rng = rng_for(22950)
    for n0, n1 in ((2, 2), (1, 3), (3, 3), (5, 1), (2, 7)):
        for dt in ("float", "half", "uint8", "cfloat"):
            a = random_view(rng, dt, (n0, n1)).permute(1, 0)
            H.check_unary("ident", a, View.empty(dt, (n1, n0)))


@pytest.mark.parametrize("dt,sc", [("cfloat", 4), ("chalf", 2), ("cdouble", 8)])
def test_complex_rows_an_odd_number_of_scalars_apart(dt, sc):
    # windows one scalar apart, rows with a gap of one scalar, a base off by one: strides that are
    # multiples of the scalar but not of the element
    rng = rng_for(22980 + sc)
    for rows, cols in ((2, 3), (6, 40), (5, 33), (37, 70)):
        for apart, shift in ((1, 0), (1, 1), (3, 0), (2 * cols + 1, 1)):
            store = random_view(rng, dt, (rows * cols * 2 + rows * 2 + 8,), specials=False)
            a = View(store.storage, dt, (rows, cols), (apart * sc, 2 * sc), shift * sc)
            print("odd complex strides", dt, rows, cols, apart, shift, flush=True)
            H.check_binary("add", a, _stored(rng, dt, (rows, cols), (1, 0), 0), View.empty(dt, (rows, cols)))
            H.check_unary("ident", a.permute(1, 0), View.empty(dt, (cols, rows)))
            H.check_binary("absgt", _stored(rng, dt, (rows, cols), (1, 0), 1), a, View.empty("bool", (rows, cols)))
