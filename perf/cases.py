"""Performance cases of the strided tensor engine: what a program has it do, through the public calls.

Every case belongs to one of ten kinds of work (the functions below are grouped by kind); the
listed cases are one or two of each at sizes that occur, and `draw` spreads over the whole range
of a kind: sizes from calls that only cost their launch to hundreds of megabytes, odd extents,
the data types and options the kind is used with.

A state holds the descriptors, outputs and workspaces that a program keeps between calls; a pass
makes the calls and nothing else.
"""
from __future__ import annotations

import ctypes
import math

import torch

import paper_1810_08723_amd as ocn

DEVICE = "cuda"
TORCH = {"bool": torch.bool, "int8": torch.int8, "uint8": torch.uint8, "int16": torch.int16, "int32": torch.int32,
         "int64": torch.int64, "half": torch.float16, "float": torch.float32, "double": torch.float64,
         "cfloat": torch.complex64, "cdouble": torch.complex128}
SIZE = {"bool": 1, "int8": 1, "uint8": 1, "int16": 2, "int32": 4, "int64": 8, "half": 2, "float": 4, "double": 8,
        "cfloat": 8, "cdouble": 16}
FLOATING = ("half", "float", "double", "cfloat", "cdouble")


def listed():
    return [
        # An add of two small tensors, one of them permuted: what a program's many small calls cost.
        {"name": "add_small", "kind": "add", "dtype": "float", "n0": 64, "n1": 48, "n2": 32},
        # A matrix plus the transpose of another, extents that are multiples of no tile.
        {"name": "add_transposed", "kind": "add", "dtype": "float", "n0": 1, "n1": 6000, "n2": 5000},
        # Integer samples times a row of factors (calibration, normalisation), odd row length.
        {"name": "scale_rows", "kind": "scale", "a": "int32", "b": "float", "out": "float", "rows": 8000, "cols": 6001},
        # Doubles to 16-bit samples, rows in reverse order, with values out of range and NaN.
        {"name": "cast_flipped", "kind": "cast", "src": "double", "dst": "int16", "rows": 4096, "cols": 4096, "swapped": False},
        # A batch of 8-bit colour images to planes of floats.
        {"name": "images_to_planes", "kind": "images", "src": "uint8", "dst": "float", "to_planes": True,
         "batch": 32, "height": 480, "width": 640, "channels": 3},
        # Complex product and magnitude mask of five-dimensional views with three different layouts.
        {"name": "complex_5d", "kind": "complex5", "s0": 16, "s1": 32, "s2": 64, "s3": 64, "s4": 8},
        # Sums over the middle axis of a batch of matrices, odd inner extent.
        {"name": "sum_middle", "kind": "reduce", "op": "sum", "dtype": "float", "out": "float", "axes": "1",
         "n0": 48, "n1": 1000, "n2": 777, "swapped": False},
        # The full sum of a large array of bytes.
        {"name": "sum_bytes", "kind": "reduce", "op": "sum", "dtype": "int8", "out": "int64", "axes": "012",
         "n0": 1, "n1": 1, "n2": 1 << 28, "swapped": False},
        # One step of Gram-Schmidt: a vector against an orthonormal basis (inner products, projection, norm).
        {"name": "project", "kind": "project", "dtype": "float", "rows": 16384, "cols": 1000},
        # An elementary function on complex numbers.
        {"name": "sine_complex", "kind": "function", "op": "sin", "dtype": "cfloat", "n": 1 << 24},
        # Rows of a table by an index array, negative indices among them.
        {"name": "take_rows", "kind": "index", "put": False, "dtype": "float", "table": 100003, "n": 65536, "width": 300},
        # The positions at which a flat array exceeds a threshold.
        {"name": "select_positions", "kind": "select", "dtype": "float", "n": 30000001},
    ]


# ---------------------------------------------------------------------------------------------
# helpers

def _generator(seed):
    return torch.Generator(device=DEVICE).manual_seed(int(seed))


def _values(gen, dtype, sizes, sigma=1.0):
    """Seeded values of a dtype: normals for the floating types (uniform in [-1, 1) would hide
    cancellation), the type's usual sample range for the integers."""
    if dtype in ("cfloat", "cdouble"):
        part = torch.float32 if dtype == "cfloat" else torch.float64
        return torch.view_as_complex(torch.randn(tuple(sizes) + (2,), generator=gen, device=DEVICE, dtype=part) * sigma)
    if dtype in ("half", "float", "double"):
        compute = torch.float64 if dtype == "double" else torch.float32
        return (torch.randn(tuple(sizes), generator=gen, device=DEVICE, dtype=compute) * sigma).to(TORCH[dtype])
    low, high = {"bool": (0, 2), "int8": (-128, 128), "uint8": (0, 256), "int16": (-30000, 30000)}.get(dtype, (-1000, 1001))
    return torch.randint(low, high, tuple(sizes), generator=gen, device=DEVICE, dtype=TORCH[dtype] if dtype != "bool"
                         else torch.uint8).to(TORCH[dtype])


def _view(t, dtype, sizes=None, strides=None, offset=0, swapped=False):
    """The engine's descriptor of a torch tensor, or of another view (strides in elements) on its storage."""
    item = SIZE[dtype]
    sizes = tuple(t.shape) if sizes is None else tuple(sizes)
    strides = t.stride() if strides is None else strides
    return ocn.Tensor(t.data_ptr(), dtype, sizes, tuple(s * item for s in strides), offset * item, t.device.index or 0, t, swapped)


def _reverse_bytes(t):
    """The same values stored in the other byte order."""
    item = t.element_size()
    return t.contiguous().view(torch.uint8).reshape(-1, item).flip(1).contiguous().view(t.dtype).reshape(t.shape)


def _wide(t):
    return t.to(torch.complex128 if t.is_complex() else torch.float64)


def _log_int(rng, low, high):
    """Log-uniform whole number; every third one rounded to a multiple of 64 where that is in range."""
    n = int(round(math.exp(rng.uniform(math.log(low), math.log(high)))))
    if n >= 128 and rng.random() < 1 / 3:
        n -= n % 64
    return min(max(n, low), high)


# ---------------------------------------------------------------------------------------------
# add: out = a + b, b a buffer [n2, n0, n1] read with its dims permuted (1, 2, 0)

def _add_inputs(case, seed):
    g = _generator(seed)
    n0, n1, n2 = case["n0"], case["n1"], case["n2"]
    return _values(g, case["dtype"], (n0, n1, n2)), _values(g, case["dtype"], (n2, n0, n1))


def _add_prepare(case, seed):
    a, b = _add_inputs(case, seed)
    out = torch.empty_like(a)
    d = case["dtype"]
    return {"a": _view(a, d), "b": _view(b.permute(1, 2, 0), d), "out": _view(out, d), "result": out}


def _add_run(s):
    ocn.binary("add", s["a"], s["b"], s["out"])
    return s["result"]


def _add_exact(case, seed):
    a, b = _add_inputs(case, seed)
    return _wide(a) + _wide(b).permute(1, 2, 0)


def _add_work(case):
    n = case["n0"] * case["n1"] * case["n2"]
    return {"bytes": 3 * n * SIZE[case["dtype"]], "flops": n * (2 if case["dtype"][0] == "c" else 1)}


def _add_draw(rng):
    dtype = rng.choice(("half", "float", "float", "double", "int32", "cfloat"))
    n = _log_int(rng, 1 << 12, (1 << 27) // SIZE[dtype])
    if rng.random() < 0.5:      # a matrix and a transposed one
        n0 = 1
        n1 = _log_int(rng, 16, max(16, n // 16))
    else:
        n0 = _log_int(rng, 2, 64)
        n1 = _log_int(rng, 8, max(8, n // n0 // 8))
    return {"dtype": dtype, "n0": n0, "n1": n1, "n2": max(1, n // n0 // n1)}


# ---------------------------------------------------------------------------------------------
# scale: out[i, j] = a[i, j] * b[j], types converted on load

def _scale_inputs(case, seed):
    g = _generator(seed)
    return _values(g, case["a"], (case["rows"], case["cols"])), _values(g, case["b"], (1, case["cols"]))


def _scale_prepare(case, seed):
    a, b = _scale_inputs(case, seed)
    out = torch.empty((case["rows"], case["cols"]), dtype=TORCH[case["out"]], device=DEVICE)
    return {"a": _view(a, case["a"]), "b": _view(b, case["b"]), "out": _view(out, case["out"]), "result": out}


def _scale_run(s):
    ocn.binary("mul", s["a"], s["b"], s["out"])
    return s["result"]


def _scale_exact(case, seed):
    a, b = _scale_inputs(case, seed)
    return _wide(a) * _wide(b)


def _scale_work(case):
    n = case["rows"] * case["cols"]
    return {"bytes": n * (SIZE[case["a"]] + SIZE[case["out"]]) + case["cols"] * SIZE[case["b"]], "flops": n}


def _scale_draw(rng):
    a, b, out = rng.choice((("int32", "float", "float"), ("float", "float", "float"), ("half", "float", "float"),
                            ("uint8", "float", "float"), ("int16", "float", "double"), ("half", "half", "half"),
                            ("double", "double", "double"), ("int32", "int32", "int32")))
    n = _log_int(rng, 1 << 12, (3 << 27) // (SIZE[a] + SIZE[out]))
    cols = _log_int(rng, 16, min(1 << 14, n))
    return {"a": a, "b": b, "out": out, "rows": max(1, n // cols), "cols": cols}


# ---------------------------------------------------------------------------------------------
# cast: a type-converting copy with the rows in reverse order, also from data in the other byte order

def _cast_inputs(case, seed):
    g = _generator(seed)
    x = _values(g, case["src"], (case["rows"], case["cols"]), 2e4)
    if case["src"] in ("float", "double"):
        x[torch.rand(x.shape, generator=g, device=DEVICE) < 1e-4] = math.nan
    return x


def _cast_prepare(case, seed):
    x = _cast_inputs(case, seed)
    rows, cols = case["rows"], case["cols"]
    if case["swapped"]:
        x = _reverse_bytes(x)
    out = torch.empty((rows, cols), dtype=TORCH[case["dst"]], device=DEVICE)
    return {"src": _view(x, case["src"], (rows, cols), (-cols, 1), (rows - 1) * cols, case["swapped"]),
            "out": _view(out, case["dst"]), "result": out}


def _cast_run(s):
    ocn.cast_copy(s["src"], s["out"])
    return s["result"]


def _cast_exact(case, seed):
    return _wide(_cast_inputs(case, seed)).flip(0) if case["dst"] in ("float", "double") else None


def _cast_work(case):
    n = case["rows"] * case["cols"]
    return {"bytes": n * (SIZE[case["src"]] + SIZE[case["dst"]]), "flops": n}


def _cast_draw(rng):
    src, dst = rng.choice((("double", "int16"), ("double", "float"), ("float", "half"), ("int16", "float"),
                           ("int32", "double"), ("float", "uint8"), ("float", "float")))
    n = _log_int(rng, 1 << 12, (3 << 26) // (SIZE[src] + SIZE[dst]))
    cols = _log_int(rng, 16, min(1 << 14, n))
    return {"src": src, "dst": dst, "rows": max(1, n // cols), "cols": cols, "swapped": rng.random() < 0.25}


# ---------------------------------------------------------------------------------------------
# images: interleaved pixels [batch, height, width, channels] to planes [batch, channels, height,
# width] or back, converting the samples

def _images_inputs(case, seed):
    b, h, w, c = case["batch"], case["height"], case["width"], case["channels"]
    g = _generator(seed)
    if case["src"] == "uint8":
        return _values(g, "uint8", (b, h, w, c) if case["to_planes"] else (b, c, h, w))
    x = torch.rand((b, h, w, c) if case["to_planes"] else (b, c, h, w), generator=g, device=DEVICE) * 255
    return x.to(TORCH[case["src"]])


def _images_prepare(case, seed):
    x = _images_inputs(case, seed)
    src = x.permute(0, 3, 1, 2) if case["to_planes"] else x.permute(0, 2, 3, 1)
    out = torch.empty(src.shape, dtype=TORCH[case["dst"]], device=DEVICE)
    return {"src": _view(src, case["src"]), "out": _view(out, case["dst"]), "result": out}


def _images_run(s):
    ocn.cast_copy(s["src"], s["out"])
    return s["result"]


def _images_exact(case, seed):
    if case["dst"] not in FLOATING:
        return None
    x = _wide(_images_inputs(case, seed))
    return x.permute(0, 3, 1, 2) if case["to_planes"] else x.permute(0, 2, 3, 1)


def _images_work(case):
    n = case["batch"] * case["height"] * case["width"] * case["channels"]
    return {"bytes": n * (SIZE[case["src"]] + SIZE[case["dst"]]), "flops": n}


def _images_draw(rng):
    src, dst = rng.choice((("uint8", "float"), ("uint8", "half"), ("float", "float"), ("float", "uint8"), ("uint8", "uint8")))
    height, width = _log_int(rng, 32, 1080), _log_int(rng, 32, 1920)
    channels = rng.choice((2, 3, 3, 3, 4))
    batch = _log_int(rng, 1, max(1, (1 << 28) // (SIZE[src] + SIZE[dst]) // (height * width * channels)))
    return {"src": src, "dst": dst, "to_planes": rng.random() < 0.5, "batch": min(batch, 256), "height": height,
            "width": width, "channels": channels}


# ---------------------------------------------------------------------------------------------
# complex5: c = a * b and mask = |a| > |b| on five-dimensional complex views; a is every other
# element along axis 2 of a permuted buffer, b row-major, c written permuted

_PERM_A, _PERM_C = (4, 2, 0, 3, 1), (3, 0, 4, 1, 2)


def _complex5_sizes(case):
    return tuple(case[f"s{i}"] for i in range(5))


def _complex5_inputs(case, seed):
    g = _generator(seed)
    s = _complex5_sizes(case)
    logical = (s[0], s[1], 2 * s[2], s[3], s[4])
    buffer = [0] * 5
    for i, p in enumerate(_PERM_A):
        buffer[p] = logical[i]
    return _values(g, "cfloat", buffer).permute(_PERM_A)[:, :, ::2], _values(g, "cfloat", s)


def _complex5_prepare(case, seed):
    a, b = _complex5_inputs(case, seed)
    s = _complex5_sizes(case)
    buffer = [0] * 5
    for i, p in enumerate(_PERM_C):
        buffer[p] = s[i]
    c = torch.empty(buffer, dtype=torch.complex64, device=DEVICE)
    mask = torch.empty(s, dtype=torch.bool, device=DEVICE)
    return {"a": _view(a, "cfloat"), "b": _view(b, "cfloat"), "c": _view(c.permute(_PERM_C), "cfloat"),
            "mask": _view(mask, "bool"), "result": [c.permute(_PERM_C), mask]}


def _complex5_run(s):
    ocn.binary("mul", s["a"], s["b"], s["c"])
    ocn.binary("absgt", s["a"], s["b"], s["mask"])
    return s["result"]


def _complex5_exact(case, seed):
    a, b = _complex5_inputs(case, seed)
    return [_wide(a) * _wide(b), None]


def _complex5_work(case):
    n = math.prod(_complex5_sizes(case))
    return {"bytes": 25 * n, "flops": 13 * n}


def _complex5_draw(rng):
    while True:
        s = [_log_int(rng, 2, 72) for _ in range(5)]
        if 1 << 10 <= math.prod(s) <= 1 << 24:
            return {f"s{i}": v for i, v in enumerate(s)}


# ---------------------------------------------------------------------------------------------
# reduce: one reduction of [n0, n1, n2] along the axes named

def _reduce_axes(case):
    return [int(c) for c in case["axes"]]


def _reduce_inputs(case, seed):
    return _values(_generator(seed), case["dtype"], (case["n0"], case["n1"], case["n2"]))


def _reduce_prepare(case, seed):
    x = _reduce_inputs(case, seed)
    kept = [n for i, n in enumerate(x.shape) if i not in _reduce_axes(case)]
    out = torch.empty(kept, dtype=TORCH[case["out"]], device=DEVICE)
    a = _view(_reverse_bytes(x) if case["swapped"] else x, case["dtype"], swapped=case["swapped"])
    o, axes = _view(out, case["out"]), _reduce_axes(case)
    need = ocn.reduce_workspace_bytes(case["op"], a, axes, o)
    return {"op": case["op"], "a": a, "axes": axes, "out": o, "result": out,
            "workspace": torch.empty(max(need, 256), dtype=torch.uint8, device=DEVICE)}


def _reduce_run(s):
    ocn.reduce(s["op"], s["a"], s["axes"], s["out"], workspace=s["workspace"])
    return s["result"]


def _reduce_exact(case, seed):
    if case["out"] not in FLOATING:
        return None
    x = _wide(_reduce_inputs(case, seed))
    return x.sum(_reduce_axes(case)) if case["op"] == "sum" else x.amax(_reduce_axes(case))


def _reduce_work(case):
    n = case["n0"] * case["n1"] * case["n2"]
    kept = math.prod(case[f"n{i}"] for i in range(3) if i not in _reduce_axes(case))
    return {"bytes": n * SIZE[case["dtype"]] + kept * SIZE[case["out"]], "flops": n}


def _reduce_draw(rng):
    op, dtype, out = rng.choice((("sum", "float", "float"), ("sum", "half", "float"), ("sum", "double", "double"),
                                 ("sum", "int8", "int64"), ("sum", "int32", "int64"), ("max", "half", "half"),
                                 ("max", "float", "float"), ("any", "bool", "bool"), ("sum", "cfloat", "cfloat")))
    n = _log_int(rng, 1 << 12, (1 << 28) // SIZE[dtype])
    n1 = _log_int(rng, 4, max(4, min(1 << 14, n // 4)))
    n2 = _log_int(rng, 1, max(1, min(1 << 14, n // n1)))
    return {"op": op, "dtype": dtype, "out": out, "axes": rng.choice(("0", "1", "2", "01", "12", "02", "012")),
            "n0": max(1, n // n1 // n2), "n1": n1, "n2": n2,
            "swapped": SIZE[dtype] > 1 and rng.random() < 0.15}


# ---------------------------------------------------------------------------------------------
# project: one step of Gram-Schmidt.  r = V^T x, p = V r, y = x - p, d = y . y, q = y / sqrt(d)

def _project_inputs(case, seed):
    g = _generator(seed)
    scale = 1.0 / math.sqrt(case["rows"])     # columns of about unit length, as a basis has
    v = _values(g, case["dtype"], (case["rows"], case["cols"]), scale)
    return v, _values(g, case["dtype"], (case["rows"], 1))


def _project_prepare(case, seed):
    v, x = _project_inputs(case, seed)
    d, m, k = case["dtype"], case["rows"], case["cols"]
    new = lambda *sizes: torch.empty(sizes, dtype=TORCH[d], device=DEVICE)  # noqa: E731
    r, p, y, dot, root, q = new(k), new(m), new(m), new(1), new(1), new(m)
    s = {"d": d, "v": _view(v, d), "x": _view(x, d), "x1": _view(x.reshape(m), d), "r": _view(r, d), "p": _view(p, d),
         "y": _view(y, d), "dot": _view(dot, d, (), ()), "root": _view(dot, d), "norm": _view(root, d), "q": _view(q, d),
         "result": {"r": r, "y": y, "norm": root, "q": q}}
    need = max(ocn.binary_reduce_workspace_bytes("mul", "sum", s["v"], s["x"], [0], s["r"], d),
               ocn.binary_reduce_workspace_bytes("mul", "sum", s["v"], s["r"], [1], s["p"], d),
               ocn.binary_reduce_workspace_bytes("mul", "sum", s["y"], s["y"], [0], s["dot"], d), 256)
    s["workspace"] = torch.empty(need, dtype=torch.uint8, device=DEVICE)
    return s


def _project_run(s):
    d, ws = s["d"], s["workspace"]
    ocn.binary_reduce("mul", "sum", s["v"], s["x"], [0], s["r"], d, workspace=ws)
    ocn.binary_reduce("mul", "sum", s["v"], s["r"], [1], s["p"], d, workspace=ws)
    ocn.binary("sub", s["x1"], s["p"], s["y"])
    ocn.binary_reduce("mul", "sum", s["y"], s["y"], [0], s["dot"], d, workspace=ws)
    ocn.unary("sqrt", s["root"], s["norm"])
    ocn.binary("div", s["y"], s["norm"], s["q"])
    return s["result"]


def _project_exact(case, seed):
    v, x = (_wide(t) for t in _project_inputs(case, seed))
    r = (v * x).sum(0)
    y = x[:, 0] - (v * r).sum(1)
    norm = y.square().sum().sqrt().reshape(1)
    return {"r": r, "y": y, "norm": norm, "q": y / norm}


def _project_work(case):
    m, k, size = case["rows"], case["cols"], SIZE[case["dtype"]]
    return {"bytes": size * (2 * m * k + 3 * m + k + 1), "flops": 4 * m * k + 4 * m}


def _project_draw(rng):
    dtype = rng.choice(("float", "float", "double"))
    n = _log_int(rng, 1 << 12, (1 << 27) // SIZE[dtype])
    cols = _log_int(rng, 4, min(4096, n // 64))
    return {"dtype": dtype, "rows": n // cols, "cols": cols}


# ---------------------------------------------------------------------------------------------
# function: an elementary function of every element of a flat array

_FUNCTIONS = {"sin": torch.sin, "cos": torch.cos, "exp": torch.exp, "log": torch.log, "tanh": torch.tanh,
              "sqrt": torch.sqrt, "atan": torch.atan, "abs": torch.abs}


def _function_inputs(case, seed):
    x = _values(_generator(seed), case["dtype"], (case["n"],), 3.0)
    return x.abs() + 1e-3 if case["op"] in ("log", "sqrt") and not x.is_complex() else x


def _function_prepare(case, seed):
    x = _function_inputs(case, seed)
    out = torch.empty_like(x)
    return {"op": case["op"], "a": _view(x, case["dtype"]), "out": _view(out, case["dtype"]), "result": out}


def _function_run(s):
    ocn.unary(s["op"], s["a"], s["out"])
    return s["result"]


def _function_exact(case, seed):
    return _FUNCTIONS[case["op"]](_wide(_function_inputs(case, seed)))


def _function_work(case):
    return {"bytes": 2 * case["n"] * SIZE[case["dtype"]], "flops": 20 * case["n"] * (4 if case["dtype"][0] == "c" else 1)}


def _function_draw(rng):
    dtype = rng.choice(("half", "float", "float", "double", "cfloat", "cdouble"))
    op = rng.choice(("sin", "cos", "exp", "log", "tanh", "sqrt", "atan"))
    return {"op": op, "dtype": dtype, "n": _log_int(rng, 1 << 10, (1 << 27) // SIZE[dtype])}


# ---------------------------------------------------------------------------------------------
# index: an index array bound to a table's rows, then the rows read ("take") or written ("put")

def _index_inputs(case, seed):
    g = _generator(seed)
    rows, n = case["table"], case["n"]
    table = _values(g, case["dtype"], (rows, case["width"]))
    if case["put"]:      # every row is written at most once
        index = torch.randperm(rows, generator=g, device=DEVICE)[:n].contiguous()
        src = _values(g, case["dtype"], (n, case["width"]))
    else:
        index = torch.randint(0, rows, (n,), generator=g, device=DEVICE)
        src = None
    negative = torch.rand((n,), generator=g, device=DEVICE) < 0.1
    return table, torch.where(negative, index - rows, index), src


def _index_prepare(case, seed):
    table, index, src = _index_inputs(case, seed)
    d, n, width = case["dtype"], case["n"], case["width"]
    offsets = torch.empty(n, dtype=torch.int64, device=DEVICE)
    s = {"put": case["put"], "index": _view(index, "int64"), "rows": case["table"], "pitch": width * SIZE[d],
         "last": (case["table"] - 1) * width * SIZE[d], "offsets": offsets, "bound": _view(offsets, "int64"),
         "invalid": torch.zeros(1, dtype=torch.int64, device=DEVICE), "inner": _view(table, d, (width,), (1,))}
    if case["put"]:
        s["src"], s["result"] = _view(src, d), [offsets, s["invalid"], table]
    else:
        out = torch.empty((n, width), dtype=TORCH[d], device=DEVICE)
        s["out"], s["result"] = _view(out, d), [offsets, s["invalid"], out]
    return s


def _index_run(s):
    ocn.index_offsets(s["index"], s["rows"], s["pitch"], s["bound"], s["invalid"])
    if s["put"]:
        ocn.scatter(s["src"], s["offsets"], 0, s["last"], s["inner"])
    else:
        ocn.gather(s["inner"], s["offsets"], 0, s["last"], s["out"])
    return s["result"]


def _index_exact(case, seed):
    table, index, src = _index_inputs(case, seed)
    if case["put"]:
        table[index] = src
        return [None, None, _wide(table)]
    return [None, None, _wide(table[index])]


def _index_work(case):
    moved = case["n"] * case["width"] * SIZE[case["dtype"]]
    return {"bytes": 2 * moved + 24 * case["n"], "flops": 0}     # index, offsets written and read, rows


def _index_draw(rng):
    dtype = rng.choice(("half", "float", "double"))
    width = rng.choice((1, _log_int(rng, 2, 1024)))
    n = _log_int(rng, 1 << 8, (1 << 26) // SIZE[dtype] // (width + 4))
    return {"put": rng.random() < 0.4, "dtype": dtype, "table": n + _log_int(rng, 1, 2 * n), "n": n, "width": width}


# ---------------------------------------------------------------------------------------------
# select: mask = x > t, then the offsets of the selected positions

def _select_inputs(case, seed):
    g = _generator(seed)
    return _values(g, case["dtype"], (case["n"],), 500.0), _values(g, case["dtype"], (1,), 100.0)


def _select_prepare(case, seed):
    x, t = _select_inputs(case, seed)
    n, d = case["n"], case["dtype"]
    mask = torch.empty(n, dtype=torch.bool, device=DEVICE)
    offsets = torch.zeros(n, dtype=torch.int64, device=DEVICE)
    count = torch.zeros(1, dtype=torch.int64, device=DEVICE)
    m = _view(mask, "bool")
    need = ocn.binding.lib().ocn_mask_offsets_workspace_bytes(ctypes.byref(m.desc()))
    workspace = torch.empty(max(need, 256), dtype=torch.uint8, device=DEVICE)
    return {"x": _view(x, d), "t": _view(t, d), "m": m, "stride": [SIZE[d]], "offsets": offsets, "count": count,
            "workspace": workspace, "result": [mask, offsets, count]}


def _select_run(s):
    ocn.binary("gt", s["x"], s["t"], s["m"])
    ocn.mask_offsets(s["m"], s["stride"], s["offsets"], s["count"], workspace=s["workspace"])
    return s["result"]


def _select_exact(case, seed):
    return None


def _select_work(case):
    # values read, mask written and read once, about half of the positions written
    return {"bytes": case["n"] * (SIZE[case["dtype"]] + 2 + 4), "flops": case["n"]}


def _select_draw(rng):
    dtype = rng.choice(("float", "float", "double", "int32"))
    return {"dtype": dtype, "n": _log_int(rng, 1 << 10, 30000000)}


# ---------------------------------------------------------------------------------------------

_KINDS = ("add", "scale", "cast", "images", "complex5", "reduce", "project", "function", "index", "select")


def draw(rng):
    kind = rng.choice(_KINDS)
    return {"kind": kind, **globals()[f"_{kind}_draw"](rng)}


def prepare(case, seed):
    return {"kind": case["kind"], **globals()[f"_{case['kind']}_prepare"](case, seed)}


def run(state):
    return _RUN[state["kind"]](state)


_RUN = {kind: globals()[f"_{kind}_run"] for kind in _KINDS}


def work(case):
    return globals()[f"_{case['kind']}_work"](case)


def exact(case, seed):
    return globals()[f"_{case['kind']}_exact"](case, seed)


def tolerance(case):
    """Copies, conversions and single arithmetic operations round once: any correct result has the
    same bits.  Elementary functions are good to a few units in the last place (complex ones
    relative to the magnitude).  Sums are accumulated in wider types (doubles in doubles) and
    differ by their final rounding, or by the order of the additions for doubles; the steps of
    a projection carry such differences on."""
    kind = case["kind"]
    if kind == "function":
        unit = {"half": 5e-4, "float": 6e-8, "cfloat": 6e-8, "double": 1.2e-16, "cdouble": 1.2e-16}[case["dtype"]]
        return {"rel": 4 * unit, "max": 64 * unit}
    if kind == "project":
        return {"rel": 5e-7, "max": 2e-5} if case["dtype"] == "float" else {"rel": 2e-14, "max": 1e-12}
    if kind == "reduce" and case["op"] == "sum" and case["out"] in FLOATING:
        return {"rel": 1e-14, "max": 1e-12} if case["dtype"] == "double" else {"rel": 2e-7, "max": 4e-6}
    return "exact"
