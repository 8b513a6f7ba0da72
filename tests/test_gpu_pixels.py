"""Copies and casts between planes and interleaved pixels: every sample type pair, two to four
channels, numbers of pixels around the vector's, padded rows, reversed planes, any alignment."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

SAMPLES = ("uint8", "uint16", "int16", "half", "float")


def _off_by(rng, dtype, shape, k):
    n = int(np.prod(shape))
    flat = random_view(rng, dtype, (n + 8,)) if rng is not None else View.empty(dtype, (n + 8,))
    es = flat.strides[0]
    strides = tuple(es * int(np.prod(shape[d + 1:])) for d in range(len(shape)))
    return View(flat.storage, dtype, tuple(shape), strides, flat.offset + k * es)


def _both_ways(rng, din, dout, c, n, h, w, k):
    print("pixels", din, dout, c, n, h, w, k, flush=True)
    H.check_unary("ident", _off_by(rng, din, (n, h, w, c), k).permute(0, 3, 1, 2), _off_by(None, dout, (n, c, h, w), k))
    H.check_unary("ident", _off_by(rng, din, (n, c, h, w), k).permute(0, 2, 3, 1), _off_by(None, dout, (n, h, w, c), k))


@pytest.mark.parametrize("din", SAMPLES)
@pytest.mark.parametrize("dout", SAMPLES)
@pytest.mark.parametrize("c", (2, 3, 4))
def test_sample_types_and_channels(din, dout, c):
    rng = rng_for(26000 + c + sum(map(ord, din + dout)))
    for n, h, w, k in ((1, 1, 3, 0), (2, 1, 4, 1), (1, 3, 7, 1), (2, 4, 8, 0), (1, 1, 16, 3), (3, 1, 17, 1), (2, 13, 41, 1), (1, 40, 64, 0)):
        _both_ways(rng, din, dout, c, n, h, w, k)


@pytest.mark.parametrize("dtype", ("int8", "bool", "int32", "uint64", "double", "cfloat", "chalf", "cdouble"))
def test_plain_copies_of_other_types(dtype):
    rng = rng_for(26500)
    for c in (2, 3, 4, 5):
        _both_ways(rng, dtype, dtype, c, 2, 9, 11, 1)


@pytest.mark.parametrize("dtype,sc", [("chalf", 2), ("cfloat", 4)])
def test_complex_copies_aligned_to_their_scalars_only(dtype, sc):
    rng = rng_for(26550 + sc)
    for c in (2, 3, 4):
        for shift in (sc, 3 * sc):
            a, out = _off_by(rng, dtype, (2, 9, 11, c), 0), _off_by(None, dtype, (2, c, 9, 11), 0)
            a = View(a.storage, dtype, a.sizes, a.strides, shift)
            out = View(out.storage, dtype, out.sizes, out.strides, shift)
            print("complex pixels", dtype, c, shift, flush=True)
            H.check_unary("ident", a.permute(0, 3, 1, 2), out)
            H.check_unary("ident", out.permute(0, 2, 3, 1), View(View.empty(dtype, (2 * 9 * 11 * c + 8,)).storage, dtype, a.sizes, a.strides, shift))


def test_padded_rows_reversed_planes_and_byte_order():
    rng = rng_for(26600)
    big = random_view(rng, "uint8", (2, 20, 33, 3))
    crop = big.slice(1, 2, 19, 1).slice(2, 1, 32, 1)                       # rows of 31 pixels with a pitch of 33
    H.check_unary("ident", crop.permute(0, 3, 1, 2), View.empty("float", (2, 3, 17, 31)))
    H.check_unary("ident", crop.permute(0, 3, 1, 2), View.empty("uint8", (2, 3, 17, 40)).slice(3, 3, 34, 1))
    planes = random_view(rng, "float", (2, 3, 17, 31))
    H.check_unary("ident", planes.flip(1).permute(0, 2, 3, 1), View.empty("half", (2, 17, 31, 3)))
    H.check_unary("ident", planes.flip(0).permute(0, 2, 3, 1), View.empty("uint8", (2, 17, 31, 3)))
    H.check_unary("ident", big.flip(3).permute(0, 3, 1, 2), View.empty("float", (2, 3, 20, 33)))    # channels reversed
    s = planes.in_other_byte_order().permute(0, 2, 3, 1)
    out = View.empty("float", (2, 17, 31, 3))
    H.check_unary("ident", s, out)                                          # out in native order: a reversing copy
    H.check_unary("ident", s, View(out.storage, out.dtype, out.sizes, out.strides, out.offset, True))


def test_many_workgroups_of_pixels():
    rng = rng_for(26700)
    _both_ways(rng, "uint8", "float", 3, 5, 211, 307, 0)
    _both_ways(rng, "float", "float", 2, 7, 128, 130, 1)


def test_stored_bools_are_zero_or_one_afterwards():
    # any byte but zero is true, and a copy writes it as 1, whichever kernel a size and alignment gets
    rng = rng_for(26800)
    for shape in ((2, 9, 11, 3), (1, 15, 15, 2), (3, 19, 23, 4), (2, 7, 6, 5)):
        n, h, w, c = shape
        for k in (0, 1):
            print("bool bytes", shape, k, flush=True)
            for flipped in (False, True):
                a = _off_by(rng, "uint8", (n, c, h, w) if flipped else shape, k)
                a = View(a.storage, "bool", a.sizes, a.strides, a.offset)
                a = a.permute(0, 2, 3, 1) if flipped else a.permute(0, 3, 1, 2)
                H.check_unary("ident", a, _off_by(None, "bool", a.sizes, k))
