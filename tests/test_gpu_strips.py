"""Reductions over dense blocks of narrow rows in strips, plain and fused: widths around a vector and that share
no factor with it, blocks that end inside a vector, groups of lanes that the last workgroup lacks, splits and
their fold, runs of columns in an output, rows a multiple of the LDS banks apart, blocks that start
anywhere, kept dims that do not merge, byte order."""
import numpy as np
import pytest

import gpu_harness as H
from test_gpu_fused import _check
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

SIZE = {"int8": 1, "int16": 2, "half": 2, "int32": 4, "float": 4, "double": 8, "int64": 8, "cfloat": 8}


def _plan(op, a, axes, out):
    import paper_1810_08723_amd as ocn
    return ocn.plan_reduce(op, ocn.Tensor(0x1000000000, a.dtype, a.sizes, a.strides, a.offset, 0, byteswapped=getattr(a, "byteswapped", False)), list(axes),
                           ocn.Tensor(0x2000000000, out.dtype, out.sizes, out.strides, out.offset, 0))


def _reduce(a, axes, passes=None):
    """Against the oracle: whole numbers and extremes exactly, complex sums (in 64 bits) to their rounding."""
    kept = [n for d, n in enumerate(a.sizes) if d not in axes]
    exact = a.dtype.startswith("int")
    for op in ("sum", "max") if exact else ("sum",) if a.dtype == "cfloat" else ("max",):
        out = View.empty("int64" if exact and op == "sum" else a.dtype, kept)
        p = _plan(op, a, axes, out)
        assert p["vec"] == 16 // SIZE[a.dtype] and (passes is None or p["passes"] == passes), (op, a.dtype, a.sizes, p)
        print("strips", op, a.dtype, a.sizes, a.strides, axes, flush=True)
        got, want = H.run_reduce(op, a, axes, out)
        if a.dtype == "cfloat":
            g, w = got.view(np.float32).astype(np.float64), want.view(np.float32).astype(np.float64)
            fin = np.isfinite(w)
            assert np.array_equal(np.isfinite(g), fin)
            assert np.all(np.abs(g[fin] - w[fin]) <= 1.2e-7 * np.abs(w[fin]) + 1e-9 * np.abs(w[fin]).max())
        else:
            assert H.storages_equal(out.dtype, got, want), (op, a.dtype, a.sizes, H.first_mismatch(out.dtype, got, want))


def _variants(rng, dtype, sizes, axis):
    """The tensor, one that starts an element into its storage, one in the other byte order, and one whose
    slowest dim keeps its distance."""
    x = random_view(rng, dtype, sizes, specials=False)
    flat = random_view(rng, dtype, (int(np.prod(sizes)) + 1,), specials=False)
    off = View(flat.storage, dtype, tuple(sizes), x.strides, flat.offset + SIZE[dtype])
    step = random_view(rng, dtype, (2 * sizes[0],) + tuple(sizes[1:]), specials=False).slice(0, 1, 2 * sizes[0], 2) if axis > 0 else x
    return [x, off, step] + ([x.in_other_byte_order()] if SIZE[dtype] > 1 and dtype != "half" else [])


@pytest.mark.parametrize("dtype", sorted(SIZE))
@pytest.mark.parametrize("rows,width", [(51, 3), (40, 2), (33, 10), (300, 5), (64, 23), (130, 100), (90, 333)])
def test_columns_of_many_blocks(dtype, rows, width):
    rng = rng_for(27000 + rows + width)
    many = -(-(2300 << 10) // (rows * width * SIZE[dtype])) + 1
    for a in _variants(rng, dtype, (many, rows, width), 1):
        _reduce(a, (1,))
    a = random_view(rng, dtype, (many // 7 + 1, rows, 7, width), specials=False).permute(0, 2, 1, 3)   # (rows apart: not a dense block)
    kept = [n for d, n in enumerate(a.sizes) if d != 2]
    out = View.empty("int64" if dtype.startswith("int") else dtype, kept)
    if dtype.startswith("int"):
        got, want = H.run_reduce("sum", a, (2,), out)
        assert H.storages_equal(out.dtype, got, want)


@pytest.mark.parametrize("dtype", ("int8", "half", "int32", "float", "double", "cfloat"))
@pytest.mark.parametrize("width", (2, 3, 8, 13, 64, 100, 250))
def test_columns_of_one_long_block(dtype, width):
    rng = rng_for(27200 + width)
    rows = (6 << 20) // (width * SIZE[dtype]) + 3
    for a in _variants(rng, dtype, (rows, width), 0):
        _reduce(a, (0,), passes=2)
    for a in _variants(rng, dtype, (3, rows // 3, width), 1):
        _reduce(a, (1,), passes=2)


@pytest.mark.parametrize("dtype", ("int8", "half", "int32", "double", "cfloat"))
@pytest.mark.parametrize("kept,inner", [(5, 3), (14, 10), (6, 33), (40, 2)])
def test_runs_of_columns(dtype, kept, inner):
    rng = rng_for(27400 + kept + inner)
    rows = (5 << 20) // (kept * inner * SIZE[dtype]) + 1
    for a in _variants(rng, dtype, (rows, kept, inner), 0):
        _reduce(a, (0, 2))


@pytest.mark.parametrize("dtype", sorted(SIZE))
@pytest.mark.parametrize("width", (2, 3, 5, 16, 22, 24, 64, 100))
def test_rows(dtype, width):
    if width * SIZE[dtype] > 1024 or (dtype == "int8" and width == 64):
        pytest.skip("not taken in strips")
    rng = rng_for(27600 + width)
    total = (13 << 20) if width % (16 // SIZE[dtype]) == 0 else (4300 << 10)
    rows = total // (width * SIZE[dtype]) + 5
    for a in _variants(rng, dtype, (3, rows // 3 + 1, width), 2)[: 4 if total < 5 << 20 else 2]:
        _reduce(a, (2,))


@pytest.mark.parametrize("dtype", ("int32", "half", "float", "double", "cfloat", "cdouble"))
@pytest.mark.parametrize("width", (2, 5, 9, 22, 37, 64, 108))
def test_products_with_a_row_and_a_column(dtype, width):
    es = 16 if dtype == "cdouble" else SIZE[dtype]
    rng = rng_for(27800 + width)
    rows = (4300 << 10) // (width * es) + 7
    v = random_view(rng, dtype, (rows, width), specials=False)
    column, row = random_view(rng, dtype, (rows, 1), specials=False), random_view(rng, dtype, (1, width), specials=False)
    other = random_view(rng, dtype, (rows, width), specials=False)
    for axis, lone in ((0, column), (1, row)):
        _check("mul", "sum", v, lone, (axis,), dtype, expect_fused=True)
        _check("sub", "sum", lone, v, (axis,), dtype, expect_fused=True)
        _check("mul", "sum", v, other, (axis,), dtype, expect_fused=True)
    if dtype in ("int32", "float", "double"):
        _check("lt", "sum", v, column, (0,), "bool", "int64")
        _check("gt", "any", row, v, (1,), "bool", "bool")
    blocks = random_view(rng, dtype, (9, rows // 9, width), specials=False)
    _check("mul", "sum", blocks, random_view(rng, dtype, (9, rows // 9, 1), specials=False), (1,), dtype)
    _check("mul", "sum", blocks, random_view(rng, dtype, (9, 1, width), specials=False), (2,), dtype)


@pytest.mark.parametrize("dtype,sizes,axes", [("float", (30001, 9), (0,)), ("int32", (1000, 51, 3), (1,)), ("half", (300001, 9), (1,)), ("double", (60001, 6, 5), (0, 2))])
def test_nan_and_infinity(dtype, sizes, axes):
    """Infinities and NaN reach their own outputs and no others."""
    rng = rng_for(27900)
    a = random_view(rng, dtype, sizes, specials=True)
    kept = [n for d, n in enumerate(sizes) if d not in axes]
    for op in ("max", "min", "any", "all"):
        out = View.empty("bool" if op in ("any", "all") else dtype, kept)
        print("strips", op, dtype, sizes, flush=True)
        got, want = H.run_reduce(op, a, axes, out)
        assert H.storages_equal(out.dtype, got, want), (op, dtype, H.first_mismatch(out.dtype, got, want))


@pytest.mark.parametrize("dtype", ("int8", "half", "int32", "double", "cfloat"))
@pytest.mark.parametrize("rows,kept,inner", [(300, 1501, 20), (620, 1300, 9), (701, 601, 13), (1000, 67, 31), (300, 9001, 2)])
def test_runs_of_columns_of_long_rows(dtype, rows, kept, inner):
    """Runs whose workgroups end inside a vector, the last one with fewer outputs, split and whole, rows apart."""
    rng = rng_for(28000 + kept + inner)
    rows = max(rows, (4300 << 10) // (kept * inner * SIZE[dtype]) + 1)
    for a in _variants(rng, dtype, (rows, kept, inner), 0)[:: 1 if rows * kept < 1 << 20 else 3]:
        _reduce(a, (0, 2))
    _reduce(random_view(rng, dtype, (2 * rows, kept, inner), specials=False).slice(0, 0, 2 * rows, 2), (0, 2))
