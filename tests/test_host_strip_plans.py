"""Which reductions over dense blocks of narrow rows go through strips: calls that the other forms take faster, and calls
that strips take faster, on both sides of each rule (no GPU needed)."""
import pytest

import paper_1810_08723_amd as ocn

ES = {"bool": 1, "int8": 1, "uint8": 1, "int16": 2, "half": 2, "int32": 4, "float": 4, "double": 8, "cfloat": 8, "cdouble": 16, "int64": 8, "uint64": 8}
SUM = {"bool": "int64", "int8": "int64", "uint8": "uint64", "int16": "int64", "int32": "int64"}
COLUMNS, ROWS, RUNS = 1, 2, 3


def _tensor(base, dtype, sizes, first=0):
    strides, acc = [], ES[dtype]
    for n in reversed(sizes):
        strides.insert(0, 0 if n == 1 else acc)
        acc *= n
    return ocn.Tensor(base << 40, dtype, tuple(sizes), tuple(strides), first * ES[dtype])


def _strip(op, dtype, sizes, axes, first=0):
    kept = [n for d, n in enumerate(sizes) if d not in axes]
    out = SUM.get(dtype, dtype) if op in ("sum", "prod") else "bool" if op in ("any", "all") else dtype
    return ocn.plan_reduce(op, _tensor(1, dtype, sizes, first), list(axes), _tensor(2, out, kept))["strip"]


def _fused(op, dtype, sizes, axis, lone, mid=None):
    other = {"row": [*sizes[:-2], 1, sizes[-1]], "column": [*sizes[:-1], 1], "block": sizes}[lone]
    kept = [n for d, n in enumerate(sizes) if d != axis]
    mid = mid or dtype
    out = _tensor(3, "int64" if mid == "bool" else dtype, kept)
    p = ocn.plan_binary_reduce(op, "sum", _tensor(1, dtype, sizes), _tensor(2, dtype, other), [axis], out, mid)
    assert p["fused"]
    return p["strip"]


@pytest.mark.parametrize("op,dtype,sizes", [("any", "bool", (253179, 18, 2)), ("sum", "half", (15673, 9, 4)), ("max", "int16", (148557, 26, 4))])
def test_rows_of_blocks_of_a_few(op, dtype, sizes):
    """A workgroup's rows come from one block: where each is left with a few dozen bytes, rows stay with lanes of their own."""
    strides = (2 * sizes[1] * sizes[2] * ES[dtype], sizes[2] * ES[dtype], ES[dtype])
    a = ocn.Tensor(1 << 40, dtype, sizes, strides)
    out = _tensor(2, "bool" if op == "any" else "int64" if op == "sum" and dtype != "half" else dtype, sizes[:2])
    assert ocn.plan_reduce(op, a, [2], out)["strip"] == 0
    sizes = (sizes[0] // 300, sizes[1] * 300, sizes[2])
    a = ocn.Tensor(1 << 40, dtype, sizes, (2 * sizes[1] * sizes[2] * ES[dtype], sizes[2] * ES[dtype], ES[dtype]))
    assert ocn.plan_reduce(op, a, [2], _tensor(2, out.dtype, sizes[:2]))["strip"] == ROWS


@pytest.mark.parametrize("op,dtype,sizes,mid,form", [("sub", "cfloat", (48969, 18, 2), None, 0), ("lt", "int32", (28070, 11, 2), "bool", 0), ("mul", "float", (15976, 21, 3), None, 0),
                                                     ("mul", "double", (792, 99, 11), None, 0), ("mul", "cfloat", (500, 1800, 3), None, ROWS), ("lt", "int32", (280, 5100, 2), "bool", ROWS)])
def test_fused_rows_of_blocks_of_a_few(op, dtype, sizes, mid, form):
    assert _fused(op, dtype, sizes, 2, "row", mid) == form


@pytest.mark.parametrize("dtype,sizes,form", [("cfloat", (91826, 3), 0), ("cfloat", (200000, 3), ROWS), ("double", (129543, 3), 0), ("int32", (88765, 2), 0), ("int32", (400000, 2), ROWS),
                                              ("cdouble", (150000, 3), 0), ("cdouble", (200000, 3), ROWS), ("double", (26434, 27), 0), ("double", (40000, 27), ROWS),
                                              ("half", (147000, 64), 0), ("half", (300000, 64), ROWS), ("float", (60000, 64), 0), ("float", (70001, 64), ROWS), ("half", (50000, 9), 0),
                                              ("half", (150000, 9), ROWS)])
def test_rows_by_size(dtype, sizes, form):
    assert _strip("max" if dtype in ("half", "int32", "float", "double") else "sum", dtype, sizes, (1,)) == form


@pytest.mark.parametrize("dtype,sizes,lone,form", [("half", (22935, 242), "row", 0), ("half", (22935, 242), "block", ROWS), ("float", (26934, 59), "row", 0), ("float", (60000, 59), "row", ROWS),
                                                   ("double", (13924, 55), "row", 0), ("double", (20000, 55), "row", ROWS)])
def test_fused_rows_by_size(dtype, sizes, lone, form):
    assert _fused("mul", dtype, sizes, 1, lone) == form


@pytest.mark.parametrize("op,dtype,sizes,form", [("sum", "int8", (249498, 17, 2), 0), ("sum", "uint8", (25146, 24, 12), 0), ("sum", "bool", (75176, 26, 8), 0), ("sum", "int8", (90000, 40, 2), COLUMNS),
                                                 ("sum", "bool", (3126, 20, 914), 0), ("sum", "double", (16, 85, 459), 0), ("sum", "float", (3, 94, 962), 0),
                                                 ("sum", "half", (9000, 24, 49), COLUMNS), ("sum", "double", (16, 8500, 59), COLUMNS), ("sum", "half", (67684, 51, 3), COLUMNS)])
def test_columns(op, dtype, sizes, form):
    assert _strip(op, dtype, sizes, (1,)) == form


@pytest.mark.parametrize("op,dtype,sizes,form", [("max", "half", (28, 119, 871), 0), ("sum", "double", (27, 62, 484), 0), ("sum", "double", (27, 62, 121), COLUMNS), ("sum", "double", (270, 62, 484), COLUMNS),
                                                 ("sum", "cdouble", (16, 31, 410), 0), ("sum", "cdouble", (20, 64, 121), COLUMNS), ("sum", "half", (10, 59, 524), COLUMNS)])
def test_columns_of_few_blocks_of_long_rows(op, dtype, sizes, form):
    assert _strip(op, dtype, sizes, (1,)) == form


@pytest.mark.parametrize("op,dtype,sizes,form", [("max", "int8", (1917, 63, 847), 0), ("max", "uint8", (672, 47, 847), 0), ("max", "bool", (672, 47, 847), COLUMNS), ("max", "uint8", (473, 461, 192), COLUMNS),
                                                 ("max", "uint8", (172, 147, 847), COLUMNS)])
def test_columns_of_many_blocks_of_compared_bytes(op, dtype, sizes, form):
    assert _strip(op, dtype, sizes, (1,)) == form


def test_columns_of_few_short_blocks_read_one_by_one():
    assert _strip("sum", "half", (616, 5, 48), (1,), first=1) == 0
    assert _strip("sum", "half", (700, 20, 42), (1,), first=1) == COLUMNS


@pytest.mark.parametrize("op,dtype,sizes,lone,form", [("mul", "float", (65, 959, 118), "column", 0), ("mul", "cdouble", (48, 196, 67), "column", 0), ("mul", "double", (71, 177, 292), "column", 0),
                                                      ("sub", "cfloat", (2, 124, 212), "column", 0), ("mul", "int32", (9, 51, 960), "block", 0), ("mul", "double", (54, 144, 199), "block", 0),
                                                      ("lt", "float", (60, 959, 118), "column", COLUMNS), ("mul", "float", (3000, 51, 10), "column", COLUMNS),
                                                      ("mul", "half", (398, 25, 18), "column", 0), ("mul", "float", (904802, 22), "column", COLUMNS)])
def test_fused_columns(op, dtype, sizes, lone, form):
    assert _fused(op, dtype, sizes, len(sizes) - 2, lone, "bool" if op == "lt" else None) == form


@pytest.mark.parametrize("op,dtype,sizes,form", [("sum", "int8", (555, 597, 16), 0), ("sum", "half", (1474, 42, 64), 0), ("max", "half", (3833, 13, 52), 0), ("sum", "int32", (17878, 4, 44), 0),
                                                 ("sum", "int32", (19330, 16, 9), COLUMNS), ("sum", "half", (10000, 42, 62), RUNS),
                                                 ("sum", "float", (1049, 7872, 8), RUNS), ("sum", "half", (957, 7281, 7), RUNS), ("sum", "double", (298, 335, 6), 0),
                                                 ("max", "bool", (295229, 2, 48), 0), ("sum", "float", (61253, 2, 70), 0), ("sum", "int32", (18000, 3, 49), 0), ("sum", "float", (234811, 3, 29), COLUMNS)])
def test_runs_of_columns(op, dtype, sizes, form):
    assert _strip(op, dtype, sizes, (0, 2)) == form
