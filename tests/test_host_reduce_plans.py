"""Launch shapes of reductions: outputs that one workgroup takes whole, and columns of a few rows (no GPU
needed)."""
import pytest

import paper_1810_08723_amd as ocn

BASE_A, BASE_B, BASE_OUT = 0x10000000000, 0x20000000000, 0x30000000000  # far apart: never dereferenced


def _plan(op, dtype, es, sizes, axis, strides=None, offset=0):
    if strides is None:
        strides, acc = [], es
        for n in reversed(sizes):
            strides.insert(0, acc)
            acc *= n
    kept = [n for d, n in enumerate(sizes) if d != axis]
    out, acc = [], es
    for n in reversed(kept):
        out.insert(0, acc)
        acc *= n
    return ocn.plan_reduce(op, ocn.Tensor(BASE_A, dtype, tuple(sizes), tuple(strides), offset, 0), [axis],
                           ocn.Tensor(BASE_OUT, dtype, tuple(kept), tuple(out), 0, 0))


@pytest.mark.parametrize("op,dtype,es,offset,whole", [("max", "half", 2, 0, 256), ("max", "half", 2, 4, 256), ("max", "half", 2, 2, 191), ("sum", "uint8", 1, 0, 256),
                                                      ("max", "uint8", 1, 1, 191), ("max", "int8", 1, 2, 191), ("max", "float", 4, 4, 256),
                                                      ("max", "double", 8, 8, 256), ("prod", "int8", 1, 0, 191), ("prod", "uint8", 1, 0, 256)])
def test_one_workgroup_reads_whole_words(op, dtype, es, offset, whole):
    """Vectors that start inside four bytes, and products of signed bytes, are left to several workgroups beyond
    192 KiB; not where the outputs are half as many as CUs."""
    for kib in (160, 190, 192, 220, 250, 300):
        p = _plan(op, dtype, es, (kib * 1024 // es,), 0, offset=offset)
        assert (p["passes"], p["block"]) == ((1, 1024) if kib <= whole else (2, 256)), (kib, p)
        many = _plan(op, dtype, es, (128, kib * 1024 // es), 1, offset=offset)
        assert (many["passes"], many["block"]) == ((1, 1024) if kib <= 256 else (2, 256)), (kib, many)


def test_one_workgroup_reads_whole_words_of_every_row():
    n = 100000
    assert _plan("max", "half", 2, (3, n), 1)["passes"] == 1
    assert _plan("max", "half", 2, (3, n), 1, strides=(2 * n + 2, 2))["passes"] == 2


@pytest.mark.parametrize("offset,passes", [(0, 1), (4, 1), (2, 2)])
def test_one_workgroup_of_a_fused_product(offset, passes):
    n = 50000
    a, b = (ocn.Tensor(base, "half", (n,), (2,), offset, 0) for base in (BASE_A, BASE_B))
    p = ocn.plan_binary_reduce("mul", "sum", a, b, [0], ocn.Tensor(BASE_OUT, "half", (), (), 0, 0), "half")
    assert p["passes"] == passes and p["fused"]
    a, b = (ocn.Tensor(base, "half", (128, n), (2 * n, 2), offset, 0) for base in (BASE_A, BASE_B))
    p = ocn.plan_binary_reduce("mul", "sum", a, b, [1], ocn.Tensor(BASE_OUT, "half", (128,), (2,), 0, 0), "half")
    assert p["passes"] == 1 and p["fused"]


@pytest.mark.parametrize("dtype,es,rows,cols,lane", [("int16", 2, 2, 335298, False), ("half", 2, 7, 480000, False), ("half", 2, 7, 600800, True), ("half", 2, 4, 724206, True),
                                                     ("float", 4, 2, 335298, True), ("int32", 4, 8, 131072, True), ("int32", 4, 9, 131072, False),
                                                     ("double", 8, 8, 65536, True), ("double", 8, 8, 65534, False)])
def test_few_rows_of_wide_columns(dtype, es, rows, cols, lane):
    """A lane per vector of columns where there are enough of them, more of the long vectors of 16 bits."""
    lanes = -(-cols // (16 // es))
    p = _plan("max", dtype, es, (rows, cols), 0)
    assert p["vec"] == 16 // es and (p["grid"] == -(-lanes // 256)) == lane, p


@pytest.mark.parametrize("dtype,es,sizes,equal", [("int32", 4, (3, 109, 24665), True), ("cfloat", 8, (230, 89, 192), True), ("double", 8, (19, 49, 3546), True),
                                                  ("float", 4, (1, 300, 33003), True), ("float", 4, (1, 1100, 40001), True), ("double", 8, (1, 2588, 13648), False),
                                                  ("double", 8, (2, 1559, 13504), False), ("float", 4, (20, 4000, 800), False)])
def test_columns_in_equal_blocks(dtype, es, sizes, equal):
    """Equal blocks of columns do not depend on how many columns and rows there are, but for long wide rows on vector boundaries."""
    p = _plan("sum" if dtype == "cfloat" else "max", dtype, es, sizes, 1)
    lanes = -(-sizes[2] * es // 16)
    assert p["kernel"] == "red_cols" and p["vec"] == 16 // es
    assert (p["split"] == 1 and all(p["grid"] != -(-lanes // c) * sizes[0] for c in (1, 2, 4, 8, 16, 32, 64))) == equal, p
