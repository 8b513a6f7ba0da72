"""Reductions and fused reductions of operands whose rows do not start on vector boundaries: row
lengths and column counts around the vector's, operands off by a few elements, every launch shape of
the column kernel (wavefronts per workgroup, split, few columns)."""
import numpy as np
import pytest

import gpu_harness as H
from workloads.values import random_view, rng_for
from workloads.views import View

pytestmark = pytest.mark.gpu

# (operation, input, output): integers and maxima are exact; sums of floats are compared against
# their rounding (accumulated in a wider type and rounded once: 1e-6 of the sum of magnitudes)
FLOATS = {"half": np.float16, "float": np.float32, "double": np.float64}
KINDS = [("sum", "int8", "int64"), ("sum", "float", "float"), ("max", "half", "half"), ("min", "double", "double"),
         ("any", "bool", "bool"), ("sum", "int32", "int64"), ("max", "uint8", "uint8")]


def _off_by(rng, dtype, shape, k):
    n = int(np.prod(shape))
    if dtype in FLOATS:     # normals: sums and products that stay in range
        flat = View.from_numpy(rng.standard_normal(n + 16).astype(FLOATS[dtype])).slice(0, k, k + n, 1)
    else:
        flat = random_view(rng, dtype, (n + 16,), specials=False).slice(0, k, k + n, 1)
    es, strides = flat.strides[0], []
    for d in range(len(shape)):
        strides.append(es * int(np.prod(shape[d + 1:])))
    return View(flat.storage, dtype, tuple(shape), tuple(strides), flat.offset)


def _same(got, want, out, a, axes):
    if out.dtype == "float":
        g, w = got.view(np.float32).astype(np.float64), want.view(np.float32).astype(np.float64)
        mag = np.abs(a.to_numpy().astype(np.float64)).sum(axis=tuple(axes)).reshape(-1)
        return bool(np.all(np.abs(g - w) <= 1e-6 * mag))
    return H.storages_equal(out.dtype, got, want)


def _check(op, a, axes, dout):
    kept = tuple(n for d, n in enumerate(a.sizes) if d not in axes)
    out = View.empty(dout, kept)
    got, want = H.run_reduce(op, a, axes, out)
    assert _same(got, want, out, a, axes), (op, a.sizes, axes)


@pytest.mark.parametrize("kind", range(len(KINDS)))
@pytest.mark.parametrize("shape,axes", [((37, 31), (1,)), ((37, 33), (1,)), ((5, 4099), (1,)), ((300, 259), (1,)), ((7001,), (0,)),
                                        ((3, 700001), (1,)), ((33, 17), (0,)), ((2049, 63), (0,)), ((700, 261), (0,)),
                                        ((5, 300, 77), (1,)), ((40, 9, 5), (0, 1)), ((6, 50, 33), (0, 2)), ((20, 3, 1027), (0,))])
def test_ragged_reductions(kind, shape, axes):
    op, din, dout = KINDS[kind]
    rng = rng_for(23000 + 100 * kind + sum(shape))
    for k in (0, 1):
        print("ragged reduction", op, din, shape, axes, k, flush=True)
        _check(op, _off_by(rng, din, shape, k), axes, dout)


@pytest.mark.parametrize("ew,red,dtype,mid", [("mul", "sum", "float", "float"), ("mul", "sum", "double", "double"),
                                              ("add", "sum", "int32", "int32"), ("gt", "sum", "float", "bool"),
                                              ("lt", "any", "int32", "bool"), ("mul", "sum", "half", "half")])
@pytest.mark.parametrize("shape,axes", [((45, 257), (1,)), ((45, 1029), (1,)), ((3, 100001), (1,)), ((70003,), (0,)),
                                        ((45, 35), (0,)), ((3001, 37), (0,)), ((600, 515), (0,))])
def test_ragged_fused_reductions(ew, red, dtype, mid, shape, axes):
    rng = rng_for(23900 + sum(shape))
    for k in (0, 1):
        a, b = _off_by(rng, dtype, shape, k), _off_by(rng, dtype, shape, 1 - k)
        others = [b]
        if len(shape) == 2:
            others += [_off_by(rng, dtype, (1, shape[1]), 1), _off_by(rng, dtype, (shape[0], 1), 1)]
        for o in others:
            kept = tuple(n for d, n in enumerate(shape) if d not in axes)
            dout = "int64" if mid == "bool" and red == "sum" else "bool" if mid == "bool" else "double" if dtype == "double" else \
                "int64" if dtype == "int32" else "float"
            out = View.empty(dout, kept)
            print("ragged fused", ew, red, dtype, shape, axes, o.sizes, flush=True)
            got, want = H.run_binary_reduce(ew, red, a, o, axes, out, mid)
            if dout in ("float", "double"):
                ft = np.float32 if dout == "float" else np.float64
                g, w = got.view(ft).astype(np.float64), want.view(ft).astype(np.float64)
                mag = np.abs(a.to_numpy().astype(np.float64) * o.to_numpy().astype(np.float64)).sum(axis=tuple(axes)).reshape(-1)
                # half products are accumulated in single precision: 1e-3, as for its plain sums
                assert np.all(np.abs(g - w) <= {"float": 1e-6, "double": 1e-13, "half": 1e-3}[dtype] * mag)
            else:
                assert np.array_equal(got, want)


def test_in_the_other_byte_order():
    rng = rng_for(23990)
    a = random_view(rng, "float", (201, 77), specials=False).in_other_byte_order()
    for axes in ((0,), (1,)):
        _check("max", a, axes, "float")


@pytest.mark.parametrize("shape", [(1000, 65537), (5000, 32767), (3000, 8193)])
def test_byte_columns_within_the_library_s_own_scratch(shape):
    # narrower column blocks instead of more splits where the partial results are bounded
    import torch
    import paper_1810_08723_amd as ocn
    x = torch.randint(-128, 128, shape, dtype=torch.int8, device="cuda:0")
    out = torch.empty(shape[1], dtype=torch.int64, device="cuda:0")
    print("byte columns", shape, flush=True)
    ocn.binding.reduce_scratch("sum", ocn.Tensor(x.data_ptr(), "int8", shape, (shape[1], 1), 0, 0, x), [0],
                               ocn.Tensor(out.data_ptr(), "int64", shape[1:], (8,), 0, 0, out))
    torch.cuda.synchronize()
    assert np.array_equal(out.cpu().numpy(), x.cpu().numpy().astype(np.int64).sum(axis=0))


MORE = KINDS + [("sum", "uint8", "uint64"), ("any", "int16", "bool"), ("all", "half", "bool"), ("min", "int16", "int16"),
                ("prod", "int32", "int64"), ("sum", "cfloat", "cfloat")]


@pytest.mark.parametrize("kind", range(len(MORE)))
@pytest.mark.parametrize("n", (32, 33, 47, 91, 131))
def test_several_reduced_dims_of_ragged_rows(kind, n):
    """Rows that end inside a vector and lie a few elements apart: every lane of a group takes whole
    vectors over several rows, the last of a row moved back to end with it."""
    op, din, dout = MORE[kind]
    rng = rng_for(23700 + 10 * kind + n)
    for shape, axes, swap in (((2400, n), (0, 1), False), ((5, 900, n), (1, 2), False), ((3, 60, 50, n), (1, 2, 3), False),
                              ((4, 700, n), (1, 2), True), ((2, 37, n), (1, 2), False)):
        wide = shape[:-1] + (n + 3,)
        if din == "cfloat":
            a = View.from_numpy((rng.integers(-9, 9, size=wide) + 1j * rng.integers(-9, 9, size=wide)).astype(np.complex64))
        elif din in FLOATS:
            a = View.from_numpy(rng.standard_normal(wide).astype(FLOATS[din]))
        else:
            a = random_view(rng, din, wide, specials=False)
        a = a.slice(len(shape) - 1, 1, n + 1, 1)
        if len(shape) == 4:
            a = a.permute(0, 2, 1, 3)                 # outer dims that do not merge
        if swap and din not in ("int8", "uint8", "bool", "cfloat"):
            a = View(a.storage, a.dtype, a.sizes, a.strides, a.offset, True)
            if din in FLOATS and op == "sum":
                continue                              # (reversed normals are no sums with a bound)
        print("several reduced dims", op, din, shape, axes, swap, flush=True)
        kept = tuple(k for d, k in enumerate(a.sizes) if d not in axes)
        out = View.empty(dout, kept)
        got, want = H.run_reduce(op, a, axes, out)
        assert _same(got, want, out, a, axes), (op, din, a.sizes, axes)
