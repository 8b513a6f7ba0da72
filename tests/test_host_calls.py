"""The binding's direct calls hand the C ABI what its own functions hand it, and leave every call in another
form, and every error, to them (no GPU needed: a callback stands in for the library)."""
import copy
import ctypes as C
import inspect
import os
import pickle
import subprocess
import sys
import weakref

import pytest

import paper_1810_08723_amd as ocn
from paper_1810_08723_amd import binding

pytestmark = pytest.mark.skipif(binding._call is None, reason="the call module is not built for this interpreter")

P, T, I32, I64, SZ = C.c_void_p, C.POINTER(binding.OcnTensor), C.c_int32, C.c_int64, C.c_size_t
AX, ST = C.POINTER(I32), C.POINTER(I64)
C_ARGS = {"unary": (C.c_int, T, T, C.c_uint32, P), "binary": (C.c_int, T, T, T, C.c_uint32, P), "cast_copy": (T, T, P),
          "reduce": (C.c_int, T, AX, I32, T, P, SZ, P), "binary_reduce": (C.c_int, C.c_int, T, T, AX, I32, T, I32, P, SZ, P),
          "index_offsets": (T, I64, I64, T, P, P), "mask_offsets": (T, ST, P, I64, P, P, SZ, P),
          "gather": (T, P, I64, I64, I64, T, P), "scatter": (T, P, I64, I64, I64, T, P)}


class Memory:
    """Stands in for a torch tensor."""
    def __init__(self, address, n):
        self.address, self.n = address, n

    def data_ptr(self):
        return self.address

    def numel(self):
        return self.n


def _tensors():
    made = [ocn.Tensor(1 << 40 + i, "float", (4 + i, 8), (32, 4), 16 * i, 0) for i in range(3)]
    for t in made:
        t.desc()
    return made


def _usual():
    a, b, o = _tensors()
    ws = Memory(1 << 50, 4096)
    return {"unary": ("sin", a, o), "binary": ("add", a, b, o), "cast_copy": (a, o), "reduce": ("max", a, [1], o, ws),
            "binary_reduce": ("mul", "sum", a, b, (0, 1), o, "double", ws), "index_offsets": (a, 7, -12, o, Memory(1 << 51, 1)),
            "mask_offsets": (a, [8, 4], Memory(1 << 52, 0), Memory(1 << 53, 1), ws), "gather": (a, Memory(1 << 52, 9), -3, 1 << 40, o),
            "scatter": (a, Memory(1 << 52, 0), 0, 5, o)}


def _seen(args):
    """What reached the C function: structs by their bytes, arrays by their first two elements, addresses as numbers."""
    out = []
    for x in args:
        if isinstance(x, T):
            out.append(bytes(x.contents))
        elif isinstance(x, (AX, ST)):
            out.append(("list", x[0]))
        else:
            out.append(0 if x is None else x)
    return out


def _direct(name, rc=0):
    record, fallback = [], []
    proto = C.CFUNCTYPE(C.c_int, *C_ARGS[name])

    @proto
    def stand_in(*args):
        record.append(_seen(args))
        return rc

    names = dict(vars(binding), _raw_stream=(lambda device: 0x5000 + device, lambda: 3))
    call = binding._call.Call(name, lambda *a, **k: fallback.append((a, k)), names, ocn.Tensor)
    call.address = C.cast(stand_in, P).value
    return call, record, fallback, stand_in


@pytest.mark.parametrize("name", sorted(C_ARGS))
def test_the_same_reaches_the_library(name, monkeypatch):
    args = _usual()[name]
    call, record, fallback, _keep = _direct(name)
    call(*args)
    call(*args, stream=77)
    params = list(inspect.signature(getattr(ocn, name)).parameters)
    call(**dict(zip(params, args)), stream=77)
    assert not fallback and len(record) == 3 and record[1] == record[2] and record[0][:-1] == record[1][:-1]
    assert record[0][-1] == 0x5003 and record[1][-1] == 77
    # what the binding's own function passes, through the same stand-in
    own = []
    proto = C.CFUNCTYPE(C.c_int, *C_ARGS[name])
    through = proto(lambda *a: own.append(_seen(a)) or 0)
    monkeypatch.setattr(binding, "_ocn_" + name, through)
    getattr(ocn, name).__wrapped__(*args, stream=77)
    assert own == [record[1]]


@pytest.mark.parametrize("name", sorted(C_ARGS))
def test_other_forms_go_to_the_function(name):
    call, record, fallback, _keep = _direct(name)
    args = list(_usual()[name])

    class Other(ocn.Tensor):
        pass

    def with_first_tensor(x):
        at = next(i for i, v in enumerate(args) if isinstance(v, ocn.Tensor))
        return args[:at] + [x] + args[at + 1:]

    listed = ocn.Tensor(1 << 40, "float", [4, 8], [32, 4])
    listed.desc()                                                              # (never one that is kept)
    plain = dict(base=1 << 40, dtype="float", sizes=(4, 8), strides=(32, 4))
    odd = [dict(base=None), dict(base=-1), dict(base=1 << 64), dict(base=1.0), dict(dtype=10), dict(dtype="no such"), dict(sizes=(4, 8.0)), dict(sizes=(4, True)),
           dict(sizes=(1,) * 9, strides=(4,) * 9), dict(strides=(32,)), dict(strides=(1 << 63, 4)), dict(offset=None), dict(offset=1 << 63), dict(device=1 << 31),
           dict(device="0"), dict(byteswapped=1), dict(byteswapped=None)]
    forms = [with_first_tensor(x) for x in (listed, Other(1 << 40, "float", (4, 8), (32, 4)), None)]
    forms += [with_first_tensor(ocn.Tensor(**dict(plain, **x))) for x in odd]
    forms += [args[:-1], args + [None] * 9]
    if isinstance(args[0], str):
        forms += [["no such"] + args[1:], [3] + args[1:]]
    if name in ("unary", "binary"):
        forms += [args + [True], args + [-1]]
    if name in ("reduce", "binary_reduce"):
        axes = 2 if name == "reduce" else 4
        forms += [args[:axes] + [x] + args[axes + 1:] for x in ([1.0], [True], iter([1]), [0] * 9, [1 << 40])]
        forms += [args[:-1] + [None]]
    for f in forms:
        call(*f)
    call(*args, stream="0")
    call(*args, no_such=1)
    call.address = 0
    call(*args)
    assert not record and len(fallback) == len(forms) + 3


def test_errors_are_the_bindings():
    call, record, fallback, _keep = _direct("binary", rc=binding.ERR["SHAPE"])
    with pytest.raises(ocn.OcnError) as e:
        call(*_usual()["binary"])
    assert e.value.code == binding.ERR["SHAPE"] and record and not fallback


def test_names_and_signatures_stay():
    for name in C_ARGS:
        f = getattr(ocn, name)
        assert f.__name__ == name and inspect.signature(f) == inspect.signature(f.__wrapped__) and f.__doc__ == f.__wrapped__.__doc__


def test_the_public_names_stay_functions():
    """What a program may do with a function, it may do with these: copy and pickle them by name, refer to them weakly,
    keep attributes on them, make methods of them and give them another body."""
    for name in C_ARGS:
        f = getattr(ocn, name)
        assert inspect.isfunction(f) and pickle.loads(pickle.dumps(f)) is f and copy.deepcopy(f) is f and weakref.ref(f)() is f
        f.note = 1
        assert f.note == 1
        del f.note

    class Holder:
        method = ocn.unary

    assert Holder().method.__self__ is not None


def test_public_functions_go_to_the_library_directly(monkeypatch):
    """... and without the interpreter's share, unless they have been given another body."""
    record = []
    stand_in = C.CFUNCTYPE(C.c_int, *C_ARGS["unary"])(lambda *a: record.append(_seen(a)) or 0)
    monkeypatch.setattr(binding, "_raw_stream", (lambda device: 0x5000 + device, lambda: 3))
    monkeypatch.setattr(binding._direct["unary"], "address", C.cast(stand_in, P).value)
    monkeypatch.setattr(binding, "_ocn_unary", lambda *a: record.append("interpreter") or 0)
    args = _usual()["unary"]
    ocn.unary(*args)
    ocn.unary(args[0], a=args[1], out=args[2], stream=5)
    assert [r[-1] for r in record] == [0x5003, 5]
    with pytest.raises(TypeError):
        ocn.unary(*args, no_such=1)
    own = ocn.unary.__code__
    try:
        ocn.unary.__code__ = _another.__code__
        assert ocn.unary(*args) == ("another", "sin")
    finally:
        ocn.unary.__code__ = own
    assert len(record) == 2


@pytest.mark.parametrize("name", sorted(C_ARGS))
@pytest.mark.parametrize("watch", (sys.setprofile, sys.settrace))
def test_profilers_and_tracers_see_the_function(name, watch, monkeypatch):
    """A program that is profiled or traced finds the call under the function's own name."""
    stand_in = C.CFUNCTYPE(C.c_int, *C_ARGS[name])(lambda *a: 0)
    monkeypatch.setattr(binding._direct[name], "address", C.cast(stand_in, P).value)
    monkeypatch.setattr(binding, "_ocn_" + name, stand_in)
    args, entered = _usual()[name], []
    before = sys.getprofile() if watch is sys.setprofile else sys.gettrace()
    watch(lambda frame, event, arg: entered.append(frame.f_code.co_name) if event == "call" else None)
    try:
        getattr(ocn, name)(*args, stream=5)
    finally:
        watch(before)
    assert entered.count(name) == 1


def _another(op, a, out, flags=0, stream=None):
    return "another", op


def test_a_module_from_other_sources_is_left_alone():
    code = ("import sys, types, inspect; sys.modules['paper_1810_08723_amd._call'] = types.ModuleType('_call')\n"
            "import paper_1810_08723_amd as ocn\n"
            "from paper_1810_08723_amd import binding\n"
            "assert binding._call is None and not binding._direct and not hasattr(ocn.unary, '__wrapped__')\n"
            "ocn.Tensor(4096, 'float', (2,), (4,)).desc()")
    subprocess.run([sys.executable, "-c", code], cwd=os.path.dirname(os.path.dirname(os.path.abspath(__file__))), check=True, timeout=300)


@pytest.mark.parametrize("name", sorted(C_ARGS))
def test_what_desc_returns_is_what_calls_read(name):
    """An edit of the struct reaches the next call, whether it goes to the library directly or through the function."""
    args = _usual()[name]
    call, record, fallback, _keep = _direct(name)
    call(*args)
    for t in (x for x in args if isinstance(x, ocn.Tensor)):
        t.desc().offset += 1 << 20
        t.desc().size[0] = 3
        assert (t.desc().offset, t._ref._obj.size[0]) == (t.offset + (1 << 20), 3)
    call(*args)
    structs = [[binding.OcnTensor.from_buffer_copy(x) for x in r if isinstance(x, bytes)] for r in record]
    assert not fallback and [t.offset for t in structs[1]] == [t.offset + (1 << 20) for t in structs[0]]
    assert all(t.size[0] == 3 for t in structs[1])


@pytest.mark.parametrize("name", sorted(C_ARGS))
def test_new_and_changed_tensors_go_directly_too(name, monkeypatch):
    """Their descriptor is the one that the binding builds, and is kept as that one is."""
    args = list(_usual()[name])
    call, record, fallback, _keep = _direct(name)
    for form in (dict(base=(1 << 64) - 16, dtype="cdouble", sizes=(5, 0, 7), strides=(-112, 1 << 62, 16), offset=-48, device=3, byteswapped=True),
                 dict(base=1 << 40, dtype="bool", sizes=(), strides=()), dict(base=0, dtype="half", sizes=(2,) * 8, strides=(2,) * 9, offset=6)):
        new = [ocn.Tensor(**form) for x in args if isinstance(x, ocn.Tensor)]
        if name == "mask_offsets":
            args[1] = [8] * 8
        put = iter(new)
        call(*[next(put) if isinstance(x, ocn.Tensor) else x for x in args])
        seen = [x for x in record[-1] if isinstance(x, bytes)]
        with monkeypatch.context() as without:
            without.setattr(binding, "_call", None)
            plain = bytes(ocn.Tensor(**form).desc())
        assert not fallback and seen == [plain] * len(new)
        assert all(bytes(t.desc()) == seen[0] and t.desc() is t.desc() for t in new)
        new[0].offset = 64
        put = iter(new)
        call(*[next(put) if isinstance(x, ocn.Tensor) else x for x in args])
        seen = [binding.OcnTensor.from_buffer_copy(x) for x in record[-1] if isinstance(x, bytes)]
        assert not fallback and [t.offset for t in seen] == [64] + [form.get("offset", 0)] * (len(new) - 1)
