"""The strip kernels by name: each call's plan has to say that they run.  Sums, products, extremes and logical reductions of
whole values that no order of the additions rounds, so that results are compared exactly; outputs reversed, with gaps
and in the other byte order; partial results in the library's own scratch memory and under a lowered launch limit;
largest and smallest bytes where packed halves are widened; fused calls with a row, a column and another block."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

NUMPY = {"bool": np.uint8, "int8": np.int8, "uint8": np.uint8, "int16": np.int16, "int32": np.int32, "half": np.float16, "float": np.float32,
         "double": np.float64, "cfloat": np.float32, "cdouble": np.float64}
SUM = {"bool": "int64", "int8": "int64", "uint8": "uint64", "int16": "int64", "int32": "int64", "half": "float", "float": "double", "double": "double",
       "cfloat": "cdouble", "cdouble": "cdouble"}
COLUMNS, ROWS, RUNS = 1, 2, 3


def _whole(rng, dtype, sizes, first=0, op="sum"):
    """Small whole numbers (bytes of the whole range; of products +-1 and a few twos), `first` elements into the storage."""
    n = int(np.prod(sizes)) + first
    parts = 2 if dtype.startswith("c") else 1
    if op == "prod":
        x = np.where(rng.integers(0, 2, n) == 1, 1, 1 if dtype in ("bool", "uint8") else -1)
        x[rng.integers(0, n, 20)] = 1 if dtype == "bool" else 2
    elif dtype == "bool":
        x = rng.integers(0, 40, n) == 0
    elif dtype in ("int8", "uint8"):
        x = rng.integers(-128, 128, n) if dtype == "int8" else rng.integers(0, 256, n)
    else:
        x = rng.integers(-8, 9, n * parts)
    x = x.astype(NUMPY[dtype])
    es = x.itemsize * parts
    strides = [es] * len(sizes)
    for d in range(len(sizes) - 2, -1, -1):
        strides[d] = strides[d + 1] * sizes[d + 1]
    return View(x.view(np.uint8), dtype, tuple(sizes), tuple(strides), first * es)


def _out(op, dtype, kept, how=""):
    dt = SUM[dtype] if op in ("sum", "prod") else "bool" if op in ("any", "all") else dtype
    if how == "gaps":
        return View.empty(dt, [2 * n for n in kept]).slice(0, 1, 2 * kept[0], 2).slice(len(kept) - 1, 0, 2 * kept[-1], 2) if len(kept) > 1 else \
            View.empty(dt, [2 * kept[0]]).slice(0, 1, 2 * kept[0], 2)
    out = View.empty(dt, kept)
    if how == "reversed":
        strides, off = list(out.strides), out.offset
        for d in range(len(kept)):
            off += (kept[d] - 1) * strides[d]
            strides[d] = -strides[d]
        return View(out.storage, dt, tuple(kept), tuple(strides), off)
    return out.in_other_byte_order() if how == "other order" and dt != "bool" else out


def _check(op, a, axes, form, out=None, how="", scratch=False):
    import paper_1810_08723_amd as ocn
    from oracle import binding as O
    kept = [n for d, n in enumerate(a.sizes) if d not in axes]
    out = _out(op, a.dtype, kept, how) if out is None else out
    dv = H.DeviceViews()
    ta, to = dv.tensor(a), dv.tensor(out)
    plan = ocn.plan_reduce(op, ta, list(axes), to)
    assert plan["strip"] == form, (op, a.dtype, a.sizes, axes, plan)
    print("strips", form, op, a.dtype, a.sizes, a.offset, axes, how, "passes", plan["passes"], flush=True)
    (ocn.reduce_scratch if scratch else ocn.reduce)(op, ta, list(axes), to)
    dv.torch.cuda.synchronize()
    got = dv.download(out)
    O.reduce(op, a, list(axes), out)
    swapped = getattr(out, "byteswapped", False)
    assert H.storages_equal(out.dtype, got, out.storage, swapped), (op, a.dtype, a.sizes, H.first_mismatch(out.dtype, got, out.storage))
    return plan


CALLS = [   # form, dtype, sizes, axes
    (COLUMNS, "half", (4001, 51, 3), (1,)), (COLUMNS, "float", (2727, 33, 10), (1,)), (COLUMNS, "double", (300, 130, 23), (1,)), (COLUMNS, "cfloat", (70, 900, 7), (1,)),
    (COLUMNS, "int16", (900, 64, 100), (1,)), (COLUMNS, "uint8", (900, 90, 33), (1,)), (COLUMNS, "int8", (3000, 40, 30), (1,)), (COLUMNS, "bool", (9000, 50, 6), (1,)),
    (COLUMNS, "cdouble", (500, 61, 5), (1,)),
    (COLUMNS, "half", (300001, 9), (0,)), (COLUMNS, "float", (60001, 22), (0,)), (COLUMNS, "double", (9001, 79), (0,)), (COLUMNS, "int8", (700001, 13), (0,)),
    (COLUMNS, "uint8", (60001, 100), (0,)), (COLUMNS, "cfloat", (50003, 13), (0,)),
    (COLUMNS, "half", (100001, 14, 5), (0, 2)), (COLUMNS, "float", (60001, 20, 3), (0, 2)), (COLUMNS, "int8", (90001, 9, 11), (0, 2)), (COLUMNS, "uint8", (30001, 40, 5), (0, 2)),
    (ROWS, "half", (300001, 5), (1,)), (ROWS, "half", (70003, 100), (1,)), (ROWS, "float", (300001, 5), (1,)), (ROWS, "float", (60001, 22), (1,)), (ROWS, "float", (70001, 64), (1,)),
    (ROWS, "double", (200003, 3), (1,)), (ROWS, "double", (30001, 37), (1,)), (ROWS, "cfloat", (30001, 33), (1,)), (ROWS, "cdouble", (200001, 3), (1,)),
    (ROWS, "int16", (3, 50001, 27), (2,)), (ROWS, "uint8", (140003, 33), (1,)), (ROWS, "int8", (100003, 100), (1,)), (ROWS, "bool", (1000003, 7), (1,)),
    (RUNS, "half", (700, 2081, 7), (0, 2)), (RUNS, "float", (701, 1301, 5), (0, 2)), (RUNS, "double", (401, 1501, 3), (0, 2)), (RUNS, "uint8", (1021, 1331, 9), (0, 2)),
    (RUNS, "int8", (1700, 1301, 3), (0, 2)), (RUNS, "bool", (1356, 1562, 5), (0, 2)), (RUNS, "cfloat", (331, 1201, 5), (0, 2))]


@pytest.mark.parametrize("form,dtype,sizes,axes", CALLS)
def test_each_form(form, dtype, sizes, axes):
    rng = rng_for(33000 + sum(sizes))
    a = _whole(rng, dtype, sizes, first=1)
    for op in ("sum",) if dtype.startswith("c") else ("sum", "max", "any"):
        _check(op, a, axes, form)
    if not dtype.startswith("c"):
        _check("prod", _whole(rng, dtype, sizes, op="prod"), axes, form)
    _check("sum", a, axes, form, scratch=True)


@pytest.mark.parametrize("form,dtype,sizes,axes", [c for c in CALLS if c[1] in ("int16", "float", "double", "uint8")])
@pytest.mark.parametrize("how", ("reversed", "gaps", "other order"))
def test_outputs_of_any_layout(form, dtype, sizes, axes, how):
    if how == "reversed" and (form != COLUMNS or len(axes) > 1):
        form = 0     # (rows, and runs, would be read backwards)
    a = _whole(rng_for(33200 + sum(sizes)), dtype, sizes)
    _check("sum", a, axes, form, how=how)
    if dtype != "uint8":
        b = a.in_other_byte_order()
        _check("sum", b, axes, form, how=how)


@pytest.mark.parametrize("form,dtype,sizes,axes", [(COLUMNS, "float", (2727, 33, 10), (1,)), (COLUMNS, "double", (9001, 79), (0,)), (RUNS, "float", (701, 1301, 5), (0, 2))])
def test_a_lowered_launch_limit(form, dtype, sizes, axes):
    """Forms whose workgroups are more than a launch may have give way, and those that fit stay."""
    from paper_1810_08723_amd import binding
    a = _whole(rng_for(33400), dtype, sizes)
    need = _check("sum", a, axes, form)["grid"]
    try:
        binding.set_max_launch_blocks(need)
        _check("sum", a, axes, form)
        binding.set_max_launch_blocks(max(need // 4, 8))
        out = _out("sum", dtype, [n for d, n in enumerate(sizes) if d not in axes])
        print("strips, fewer workgroups", dtype, sizes, flush=True)
        got, want = H.run_reduce("sum", a, axes, out)
        assert H.storages_equal(out.dtype, got, want)
    finally:
        binding.set_max_launch_blocks(0)


@pytest.mark.parametrize("dtype", ("bool", "int8", "uint8"))
@pytest.mark.parametrize("width", (64, 256, 1024))
def test_byte_rows_a_multiple_of_the_banks_apart(dtype, width):
    """Lanes start such rows at different words; strips take them from 48 MB on."""
    rng = rng_for(33600 + width)
    a = _whole(rng, dtype, ((48 << 20) // width + 3, width))
    for op in ("sum", "max", "min", "all"):
        _check(op, a, (1,), ROWS)


@pytest.mark.parametrize("dtype,value", [("uint8", 255), ("int8", -128), ("int8", 127)])
@pytest.mark.parametrize("extra", (-1, 0, 1))
def test_saturated_byte_columns(dtype, value, extra):
    """Sums of columns in packed halves: 255, 256 and 257 rows for every wavefront (rows all at one address), in one
    launch and in splits; and in strips."""
    import paper_1810_08723_amd as ocn
    byte = np.array(value, NUMPY[dtype]).view(np.uint8)
    for width, splits in ((1 << 18, 1), (1 << 14, 16), (1 << 10, 256)):
        rows = (256 + extra) * 16 * splits
        a = View(np.full(width, byte), dtype, (rows, width), (0, 1), 0)
        out = _out("sum", dtype, [width])
        dv = H.DeviceViews()
        ta, to = dv.tensor(a), dv.tensor(out)
        p = ocn.plan_reduce("sum", ta, [0], to)
        # a workgroup of sixteen wavefronts per 64 lanes of sixteen columns and split
        assert (p["kernel"], p["strip"], p["vec"], p["block"], p["split"], p["grid"]) == ("red_cols", 0, 16, 1024, splits, width // 1024 * splits), p
        print("saturated", dtype, value, rows, width, flush=True)
        ocn.reduce("sum", ta, [0], to)
        dv.torch.cuda.synchronize()
        assert np.all(dv.download(out).view(np.int64) == value * rows)
    strip = View(np.full(70001 * 100, byte), dtype, (70000 + extra, 100), (100, 1), 0)
    _check("sum", strip, (0,), COLUMNS)


@pytest.mark.parametrize("dtype,width", [("float", 22), ("half", 9), ("double", 5), ("int32", 37), ("cfloat", 11), ("cdouble", 3)])
@pytest.mark.parametrize("lone", ("row", "column", "block"))
def test_fused_forms(dtype, width, lone):
    import paper_1810_08723_amd as ocn
    from oracle import binding as O
    rng = rng_for(33800 + width)
    es = {"half": 2, "float": 4, "int32": 4, "double": 8, "cfloat": 8, "cdouble": 16}[dtype]
    rows = (13 << 20) // (width * es) + 3
    v = _whole(rng, dtype, (rows, width), first=1)
    other = _whole(rng, dtype, {"row": (1, width), "column": (rows, 1), "block": (rows, width)}[lone])
    for axis in ((0,), (1,)):
        if (lone, axis) in (("row", (0,)), ("column", (1,))):
            continue     # (an element of the row per column: one operand's elements do not lie along the fold)
        out = _out("sum", dtype, [width if axis == (0,) else rows])
        for ew in ("mul", "sub"):
            dv = H.DeviceViews()
            ta, tb, to = dv.tensor(v), dv.tensor(other), dv.tensor(out)
            plan = ocn.plan_binary_reduce(ew, "sum", ta, tb, list(axis), to, dtype)
            if not (dtype.startswith("half") and lone == "row" and width < 8):
                assert plan["fused"] and plan["strip"] == (COLUMNS if axis == (0,) else ROWS), (ew, dtype, lone, axis, plan)
            print("strips fused", ew, dtype, v.sizes, lone, axis, flush=True)
            ocn.binary_reduce(ew, "sum", ta, tb, list(axis), to, dtype)
            dv.torch.cuda.synchronize()
            got = dv.download(out)
            O.binary_reduce(ew, "sum", v, other, list(axis), out, dtype)
            assert H.storages_equal(out.dtype, got, out.storage), (ew, dtype, lone, axis, H.first_mismatch(out.dtype, got, out.storage))
