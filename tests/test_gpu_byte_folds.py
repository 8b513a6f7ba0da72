"""Reductions of one-byte elements folded in words: rows whose ends share a word with their neighbours, of one
word and less, a multiple of the LDS banks apart; any and all over columns that end inside a vector, with few and
many rows, split and whole, in strips; and reductions over axes of one element, of every element size."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

OPS = ("any", "all", "min", "max", "sum", "prod")


def _bytes(rng, dtype, sizes, first=0):
    """Values of the whole range, and lines of the first axis that are all zero or have no zero."""
    n = int(np.prod(sizes))
    x = rng.integers(0, 2 if dtype == "bool" else 256, size=n + first, dtype=np.uint8)
    body = x[first:].reshape(sizes)
    for axis in range(len(sizes)):
        lines = np.moveaxis(body, axis, 0)
        lines[::7] = 0
        lines[3::7] = 1 if dtype == "bool" else 128
    strides = [1] * len(sizes)
    for d in range(len(sizes) - 2, -1, -1):
        strides[d] = strides[d + 1] * sizes[d + 1]
    return View(x, dtype, tuple(sizes), tuple(strides), first)


def _reduce(a, axes, ops=OPS):
    kept = [n for d, n in enumerate(a.sizes) if d not in axes]
    for op in ops:
        if a.dtype == "bool" and op in ("sum", "prod"):
            out = View.empty("int64", kept)
        else:
            out = View.empty("bool" if op in ("any", "all") else a.dtype if op in ("min", "max") else "int64", kept)
        print("bytes", op, a.dtype, a.sizes, a.offset, axes, flush=True)
        got, want = H.run_reduce(op, a, axes, out)
        assert H.storages_equal(out.dtype, got, want), (op, a.dtype, a.sizes, H.first_mismatch(out.dtype, got, want))


@pytest.mark.parametrize("dtype", ("bool", "int8", "uint8"))
@pytest.mark.parametrize("width", (2, 3, 4, 7, 31, 33, 64, 65, 100, 127, 128, 255, 256, 1000, 1024))
def test_rows(dtype, width):
    rng = rng_for(31000 + width)
    rows = (4300 << 10) // width + 3
    _reduce(_bytes(rng, dtype, (rows, width), first=width % 5), (1,), OPS if width in (3, 33, 256, 1000) else ("all", "max", "sum"))
    _reduce(_bytes(rng, dtype, (5, rows // 5 + 1, width)).slice(0, 0, 5, 2), (2,), ("any", "min", "sum"))


@pytest.mark.parametrize("dtype", ("bool", "int8", "uint8"))
@pytest.mark.parametrize("rows,width", [(1, 16), (2, 17), (9, 72), (222, 2382), (3840, 72), (60000, 20), (7, 5000), (130, 1030), (40000, 129)])
def test_columns(dtype, rows, width):
    rng = rng_for(31200 + rows + width)
    ops = ("any", "all", "min", "max")
    _reduce(_bytes(rng, dtype, (rows, width), first=rows % 3), (0,), ops)
    if rows < 1000:
        _reduce(_bytes(rng, dtype, (6, rows, width)).permute(1, 0, 2), (0,), ops)


@pytest.mark.parametrize("dtype", ("bool", "int8"))
@pytest.mark.parametrize("rows,width", [(300, 5), (33, 10), (90, 333), (51, 3)])
def test_columns_of_many_blocks(dtype, rows, width):
    rng = rng_for(31400 + rows)
    many = (2300 << 10) // (rows * width) + 2
    _reduce(_bytes(rng, dtype, (many, rows, width), first=1), (1,), ("any", "all", "min", "max"))
    _reduce(_bytes(rng, dtype, (many * rows // 7, 7, width)), (0,), ("any", "all"))


@pytest.mark.parametrize("dtype", ("bool", "int8"))
@pytest.mark.parametrize("sizes", [(1700, 301, 9), (2100, 67, 31)])
def test_runs_of_columns(dtype, sizes):
    _reduce(_bytes(rng_for(31500), dtype, sizes, first=3), (0, 2), ("any", "all", "min", "max"))


@pytest.mark.parametrize("dtype", ("bool", "uint8", "half", "float", "double", "cfloat", "cdouble"))
def test_axes_of_one_element(dtype):
    rng = rng_for(31600)
    es = {"bool": 1, "uint8": 1, "half": 2, "float": 4, "double": 8, "cfloat": 8, "cdouble": 16}[dtype]
    n = (1200 << 10) // es
    ops = ("sum", "any") if dtype.startswith("c") else ("sum", "max", "all")
    # (finite values: the oracle's compensated sums turn an infinity into NaN)
    for a in (random_view(rng, dtype, (n, 1, 3), specials=False), random_view(rng, dtype, (n // 2, 1, 2, 3), specials=False).slice(0, 1, n // 2, 1),
              random_view(rng, dtype, (3, n, 1), specials=False).slice(1, 0, n - 1, 1)):
        axis = a.sizes.index(1)
        for op in ops:
            kept = [s for d, s in enumerate(a.sizes) if d != axis]
            out = View.empty("bool" if op in ("any", "all") else "int64" if es == 1 and op == "sum" else dtype, kept)
            print("one element", op, dtype, a.sizes, flush=True)
            got, want = H.run_reduce(op, a, (axis,), out)
            assert H.storages_equal(out.dtype, got, want), (op, dtype, a.sizes, H.first_mismatch(out.dtype, got, want))
