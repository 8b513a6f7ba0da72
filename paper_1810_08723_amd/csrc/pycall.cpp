// The calls of the Python binding without its interpreter work: callables that take the arguments of
// the binding's own functions in their usual form (a Tensor of plain fields, an operation by its
// name, axes as plain ints, the current stream) straight to the C ABI, and hand every other call, and
// every error, to the function they stand for.  The public names stay the Python functions that they
// are, for whatever a program does with a function besides calling it: what serve() changes is where
// the interpreter enters them.
//
// A small call is bound by the host: sines of 3000 floats took 4.0 us a call, of which HIP's launch takes 2.4 to 3.5
// (with the machine; 1.3 for a kernel without arguments) and the plan 0.1; the rest was the interpreter and
// the argument conversions of ctypes.  3.05 us so, the six calls of a small projection 33 -> 21.4, where its
// kernels by themselves take 18.5.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstring>

#include "../../include/ocn.h"

namespace {

// what the binding expects of this module, counted up with every change to it (binding.py has the same number)
constexpr int kInterface = 3;

enum Kind { UNARY, BINARY, CAST_COPY, REDUCE, BINARY_REDUCE, INDEX_OFFSETS, MASK_OFFSETS, GATHER, SCATTER, KINDS };
// the parameters of each, in order; the last one is the stream, and those from `needed` on may be left out
struct Shape { const char *name; int needed, total; const char *params[9]; };
const Shape kShapes[KINDS] = {
    {"unary", 3, 5, {"op", "a", "out", "flags", "stream"}},
    {"binary", 4, 6, {"op", "a", "b", "out", "flags", "stream"}},
    {"cast_copy", 2, 3, {"src", "dst", "stream"}},
    {"reduce", 4, 6, {"op", "a", "axes", "out", "workspace", "stream"}},
    {"binary_reduce", 7, 9, {"ew_op", "red_op", "a", "b", "axes", "out", "mid_dtype", "workspace", "stream"}},
    {"index_offsets", 5, 6, {"index", "dim_size", "stride_bytes", "offsets", "invalid_count", "stream"}},
    {"mask_offsets", 4, 6, {"mask", "target_strides", "offsets", "count", "workspace", "stream"}},
    {"gather", 5, 6, {"a_inner", "offsets", "lo", "hi", "out", "stream"}},
    {"scatter", 5, 6, {"src", "offsets", "lo", "hi", "out_inner", "stream"}},
};
PyObject *g_params[KINDS][9];   // the same, interned
PyObject *s_direct, *s_desc, *s_raw_stream, *s_data_ptr, *s_numel, *s_check, *s_unary, *s_binary, *s_reduce, *s_dtype;
PyObject *s_ref, *s_base, *s_dtype_field, *s_sizes, *s_strides, *s_offset, *s_device, *s_byteswapped;   // of a Tensor

// ---- a descriptor that belongs to a Tensor: memory that its ctypes structure lies on -------
struct Desc {
  PyObject_HEAD
  ocn_tensor t;
};
PyTypeObject DescType = {PyVarObject_HEAD_INIT(nullptr, 0) "_call.Desc"};

int desc_buffer(PyObject *self, Py_buffer *view, int flags) {
  return PyBuffer_FillInfo(view, self, &((Desc *)self)->t, (Py_ssize_t)sizeof(ocn_tensor), 0, flags);
}
PyBufferProcs desc_as_buffer = {desc_buffer, nullptr};

bool plain_int(PyObject *o, long long *out) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  *out = PyLong_AsLongLongAndOverflow(o, &over);
  return over == 0;
}

// The descriptor of a Tensor out of its fields (its dictionary), as the binding builds it; null, with no error set,
// where they are not plain values within the struct's ranges and the binding has its own say.  (Building it there,
// field by field through ctypes, took three quarters of a call with new tensors: a binary call with three of them
// 8.3 us without this module, 10 with one that only served built ones, 2.5 so; with a library that does nothing.)
Desc *describe(PyObject *fields, PyObject *dtypes) {
  PyObject *sizes = PyDict_GetItemWithError(fields, s_sizes), *strides = PyDict_GetItemWithError(fields, s_strides);
  if (!sizes || !strides || !PyTuple_CheckExact(sizes) || !PyTuple_CheckExact(strides)) return nullptr;   // (a list may change: never kept)
  const Py_ssize_t ndim = PyTuple_GET_SIZE(sizes);
  if (ndim > OCN_MAX_DIMS || PyTuple_GET_SIZE(strides) < ndim) return nullptr;
  ocn_tensor t;
  std::memset(&t, 0, sizeof t);
  long long x;
  auto field = [&](PyObject *name) {
    PyObject *o = PyDict_GetItemWithError(fields, name);
    return o && plain_int(o, &x);
  };
  PyObject *base = PyDict_GetItemWithError(fields, s_base);
  if (!base || !PyLong_CheckExact(base)) return nullptr;
  t.base = (void *)PyLong_AsUnsignedLongLong(base);
  if (PyErr_Occurred()) {   // (negative, or more than an address)
    PyErr_Clear();
    return nullptr;
  }
  if (!field(s_offset)) return nullptr;
  t.offset = x;
  PyObject *dtype = PyDict_GetItemWithError(fields, s_dtype_field);
  PyObject *code = dtype && PyUnicode_CheckExact(dtype) ? PyDict_GetItemWithError(dtypes, dtype) : nullptr;
  if (!code || !plain_int(code, &x)) return nullptr;
  t.dtype = (int32_t)x;
  t.ndim = (int32_t)ndim;
  for (Py_ssize_t d = 0; d < ndim; ++d) {
    if (!plain_int(PyTuple_GET_ITEM(sizes, d), &x)) return nullptr;
    t.size[d] = x;
    if (!plain_int(PyTuple_GET_ITEM(strides, d), &x)) return nullptr;
    t.stride[d] = x;
  }
  if (!field(s_device) || x != (int32_t)x) return nullptr;
  t.device = (int32_t)x;
  PyObject *swapped = PyDict_GetItemWithError(fields, s_byteswapped);
  if (swapped != Py_True && swapped != Py_False) return nullptr;
  t.byteswapped = swapped == Py_True;
  Desc *d = PyObject_New(Desc, &DescType);
  if (!d) PyErr_Clear();
  else d->t = t;
  return d;
}
PyObject *module_describe(PyObject *, PyObject *const *args, Py_ssize_t n) {
  if (n != 2 || !PyDict_CheckExact(args[0]) || !PyDict_CheckExact(args[1])) {
    PyErr_SetString(PyExc_TypeError, "describe(fields, dtypes)");
    return nullptr;
  }
  Desc *d = describe(args[0], args[1]);
  if (!d) Py_RETURN_NONE;
  return (PyObject *)d;
}

// ---- a call -------------------------------------------------------------------------------
struct Call {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  int kind;
  void *address;          // of the C function; null until the library is loaded
  PyObject *function;     // what this stands for
  PyObject *globals;      // the binding's
  PyTypeObject *tensor;   // its Tensor
  PyObject *body, *defaults;   // of the function it serves, as they were
};

PyTypeObject CallType = {PyVarObject_HEAD_INIT(nullptr, 0) "_call.Call"};

// the descriptor of an argument, built and kept by the first call that takes the tensor, or null (no error set): not a
// plain Tensor, or one with fields in another form
const ocn_tensor *descriptor(const Call *c, PyObject *o) {
  if (Py_TYPE(o) != c->tensor) return nullptr;
  PyObject **dict = _PyObject_GetDictPtr(o);
  if (!dict || !*dict) return nullptr;
  PyObject *d = PyDict_GetItemWithError(*dict, s_desc);
  if (d) return Py_TYPE(d) == &DescType ? &((Desc *)d)->t : nullptr;
  PyObject *dtypes = PyDict_GetItemWithError(c->globals, s_dtype);
  if (!dtypes || !PyDict_CheckExact(dtypes) || PyDict_GetItemWithError(*dict, s_ref)) return nullptr;
  Desc *made = describe(*dict, dtypes);
  if (!made) return nullptr;
  const bool kept = PyDict_SetItem(*dict, s_desc, (PyObject *)made) == 0;
  Py_DECREF(made);
  if (!kept) PyErr_Clear();
  return kept ? &made->t : nullptr;
}
// a code out of one of the binding's dictionaries (by the name of a global)
bool code(const Call *c, PyObject *table, PyObject *name, int *out) {
  if (!PyUnicode_CheckExact(name)) return false;
  PyObject *d = PyDict_GetItemWithError(c->globals, table);
  PyObject *v = d && PyDict_CheckExact(d) ? PyDict_GetItemWithError(d, name) : nullptr;
  if (!v || !PyLong_CheckExact(v)) return false;
  *out = (int)PyLong_AsLong(v);
  return true;
}
bool plain_ints(PyObject *o, int most, long long *out, int *n) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return false;
  const Py_ssize_t len = PySequence_Fast_GET_SIZE(o);
  if (len > most) return false;
  for (Py_ssize_t i = 0; i < len; ++i)
    if (!plain_int(PySequence_Fast_GET_ITEM(o, i), out + i)) return false;
  *n = (int)len;
  return true;
}
// what a method of a torch tensor without arguments gives
bool method_int(PyObject *o, PyObject *name, long long *out) {
  PyObject *v = PyObject_CallMethodNoArgs(o, name);
  if (!v) return false;
  const bool ok = plain_int(v, out);
  Py_DECREF(v);
  return ok;
}
// the handle of the current stream; false where the binding has yet to find out how to ask for it
bool current_stream(const Call *c, void **out) {
  PyObject *raw = PyDict_GetItemWithError(c->globals, s_raw_stream);
  if (!raw || !PyTuple_CheckExact(raw) || PyTuple_GET_SIZE(raw) != 2) return false;
  PyObject *get_stream = PyTuple_GET_ITEM(raw, 0), *get_device = PyTuple_GET_ITEM(raw, 1);
  Py_INCREF(get_stream);
  PyObject *device = PyObject_CallNoArgs(get_device);
  PyObject *handle = device ? PyObject_CallOneArg(get_stream, device) : nullptr;
  Py_XDECREF(device);
  Py_DECREF(get_stream);
  bool ok = false;
  if (handle && PyLong_CheckExact(handle)) {
    *out = (void *)PyLong_AsUnsignedLongLong(handle);
    ok = !PyErr_Occurred();
  }
  Py_XDECREF(handle);
  return ok;
}

// Makes the call; false (no error set, nothing done) where the arguments are not in the usual form.
bool direct(const Call *c, PyObject *const *v, int *rc) {
  const Shape &shape = kShapes[c->kind];
  for (int i = 0; i < shape.needed; ++i)
    if (!v[i]) return false;
  // (a workspace that the function is to find: nothing else is looked at)
  const int memory = c->kind == REDUCE || c->kind == MASK_OFFSETS ? 4 : c->kind == BINARY_REDUCE ? 7 : -1;
  if (memory >= 0 && (!v[memory] || v[memory] == Py_None)) return false;
  // (copied while the interpreter is ours: another thread may replace a Tensor's descriptor meanwhile)
  ocn_tensor t[3];
  auto take = [&](int slot, int arg) {
    const ocn_tensor *d = descriptor(c, v[arg]);
    if (d) t[slot] = *d;
    return d != nullptr;
  };
  void *stream = nullptr;
  PyObject *given = v[shape.total - 1];
  auto find_stream = [&] {
    if (!given || given == Py_None) return current_stream(c, &stream);
    long long handle;
    if (!plain_int(given, &handle)) return false;
    stream = (void *)(intptr_t)handle;
    return true;
  };
  int op = 0, op2 = 0, mid = 0, naxes = 0;
  long long list[OCN_MAX_DIMS], flags = 0, x = 0, y = 0, p = 0, q = 0, r = 0, n = 0;
  int32_t axes[OCN_MAX_DIMS];
  auto find_axes = [&](PyObject *o) {
    if (!plain_ints(o, OCN_MAX_DIMS, list, &naxes)) return false;
    for (int i = 0; i < naxes; ++i) {
      if (list[i] != (int32_t)list[i]) return false;
      axes[i] = (int32_t)list[i];
    }
    return true;
  };
  auto find_flags = [&](PyObject *o) { return !o || (plain_int(o, &flags) && flags >= 0 && flags <= 0xffffffffll); };
  auto find_memory = [&](PyObject *o) { return method_int(o, s_data_ptr, &p) && method_int(o, s_numel, &n); };
  switch (c->kind) {
    case UNARY: {
      if (!code(c, s_unary, v[0], &op) || !take(0, 1) || !take(1, 2) || !find_flags(v[3]) || !find_stream()) return false;
      auto f = (int (*)(int, const ocn_tensor *, const ocn_tensor *, uint32_t, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(op, &t[0], &t[1], (uint32_t)flags, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case BINARY: {
      if (!code(c, s_binary, v[0], &op) || !take(0, 1) || !take(1, 2) || !take(2, 3) || !find_flags(v[4]) || !find_stream()) return false;
      auto f = (int (*)(int, const ocn_tensor *, const ocn_tensor *, const ocn_tensor *, uint32_t, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(op, &t[0], &t[1], &t[2], (uint32_t)flags, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case CAST_COPY: {
      if (!take(0, 0) || !take(1, 1) || !find_stream()) return false;
      auto f = (int (*)(const ocn_tensor *, const ocn_tensor *, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(&t[0], &t[1], stream);
      Py_END_ALLOW_THREADS return true;
    }
    case REDUCE: {
      if (!code(c, s_reduce, v[0], &op) || !take(0, 1) || !find_axes(v[2]) || !take(1, 3) || !find_memory(v[4]) || !find_stream()) return false;
      auto f = (int (*)(int, const ocn_tensor *, const int32_t *, int32_t, const ocn_tensor *, void *, size_t, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(op, &t[0], axes, naxes, &t[1], (void *)(intptr_t)p, (size_t)n, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case BINARY_REDUCE: {
      if (!code(c, s_binary, v[0], &op) || !code(c, s_reduce, v[1], &op2) || !take(0, 2) || !take(1, 3) || !find_axes(v[4]) || !take(2, 5) ||
          !code(c, s_dtype, v[6], &mid) || !find_memory(v[7]) || !find_stream())
        return false;
      auto f = (int (*)(int, int, const ocn_tensor *, const ocn_tensor *, const int32_t *, int32_t, const ocn_tensor *, int32_t, void *, size_t,
                        void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(op, op2, &t[0], &t[1], axes, naxes, &t[2], mid, (void *)(intptr_t)p, (size_t)n, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case INDEX_OFFSETS: {
      if (!take(0, 0) || !plain_int(v[1], &x) || !plain_int(v[2], &y) || !take(1, 3) || !method_int(v[4], s_data_ptr, &p) || !find_stream()) return false;
      auto f = (int (*)(const ocn_tensor *, int64_t, int64_t, const ocn_tensor *, void *, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(&t[0], x, y, &t[1], (void *)(intptr_t)p, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case MASK_OFFSETS: {
      if (!take(0, 0) || !plain_ints(v[1], OCN_MAX_DIMS, list, &naxes) || !method_int(v[2], s_numel, &x) || !method_int(v[2], s_data_ptr, &q) ||
          !method_int(v[3], s_data_ptr, &r) || !find_memory(v[4]) || !find_stream())
        return false;
      if (naxes < t[0].ndim) return false;   // (the other way reads past a short list as well: left to it)
      int64_t strides[OCN_MAX_DIMS];
      for (int i = 0; i < naxes; ++i) strides[i] = list[i];
      auto f = (int (*)(const ocn_tensor *, const int64_t *, void *, int64_t, void *, void *, size_t, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(&t[0], strides, x ? (void *)(intptr_t)q : nullptr, x, (void *)(intptr_t)r, (void *)(intptr_t)p, (size_t)n, stream);
      Py_END_ALLOW_THREADS return true;
    }
    case GATHER:
    case SCATTER: {
      if (!take(0, 0) || !method_int(v[1], s_numel, &n) || !method_int(v[1], s_data_ptr, &p) || !plain_int(v[2], &x) || !plain_int(v[3], &y) ||
          !take(1, 4) || !find_stream())
        return false;
      auto f = (int (*)(const ocn_tensor *, void *, int64_t, int64_t, int64_t, const ocn_tensor *, void *))c->address;
      Py_BEGIN_ALLOW_THREADS *rc = f(&t[0], n ? (void *)(intptr_t)p : nullptr, n, x, y, &t[1], stream);
      Py_END_ALLOW_THREADS return true;
    }
  }
  return false;
}

// The call if it is in the usual form (its result, or null with the error set), else `usual` is false and nothing is done.
PyObject *call_direct(const Call *c, PyObject *const *args, size_t nargsf, PyObject *kwnames, bool &usual) {
  const Shape &shape = kShapes[c->kind];
  const Py_ssize_t n = PyVectorcall_NARGS(nargsf), nkw = kwnames ? PyTuple_GET_SIZE(kwnames) : 0;
  PyObject *v[9] = {nullptr};
  usual = c->address && n <= shape.total;
  for (Py_ssize_t i = 0; usual && i < n; ++i) v[i] = args[i];
  for (Py_ssize_t k = 0; usual && k < nkw; ++k) {
    int at = 0;
    while (at < shape.total && PyTuple_GET_ITEM(kwnames, k) != g_params[c->kind][at]) ++at;
    if (at == shape.total || v[at]) usual = false;
    else v[at] = args[n + k];
  }
  int rc = 0;
  usual = usual && direct(c, v, &rc);
  if (!usual) {
    PyErr_Clear();   // (what the function finds wrong itself it says itself)
    return nullptr;
  }
  if (rc == 0) Py_RETURN_NONE;
  PyObject *check = PyDict_GetItemWithError(c->globals, s_check), *code_ = check ? PyLong_FromLong(rc) : nullptr;
  if (!code_) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, "the binding's _check is gone");
    return nullptr;
  }
  PyObject *none = PyObject_CallOneArg(check, code_);   // raises
  Py_DECREF(code_);
  return none;
}

PyObject *call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
  bool usual;
  PyObject *result = call_direct((Call *)self, args, nargsf, kwnames, usual);
  return usual ? result : PyObject_Vectorcall(((Call *)self)->function, args, nargsf & ~PY_VECTORCALL_ARGUMENTS_OFFSET, kwnames);
}

// Where the interpreter enters a function that is served; its Call is an attribute of the function.  A thread
// that is profiled or traced sees the function's own frame.
vectorcallfunc g_interpret;   // where it enters any other
PyObject *function_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
  const PyFunctionObject *f = (PyFunctionObject *)self;
  const PyThreadState *thread = PyThreadState_Get();
  Call *c = f->func_dict && !thread->c_profilefunc && !thread->c_tracefunc ? (Call *)PyDict_GetItemWithError(f->func_dict, s_direct) : nullptr;
  if (c && Py_TYPE(c) == &CallType && f->func_code == c->body && f->func_defaults == c->defaults) {   // (no other body given)
    bool usual;
    Py_INCREF(c);
    PyObject *result = call_direct(c, args, nargsf, kwnames, usual);
    Py_DECREF(c);
    if (usual) return result;
  }
  return g_interpret(self, args, nargsf, kwnames);
}
PyObject *call_serve(PyObject *self, PyObject *function) {
  if (!PyFunction_Check(function)) {
    PyErr_SetString(PyExc_TypeError, "not a Python function");
    return nullptr;
  }
  PyFunctionObject *f = (PyFunctionObject *)function;
  Call *c = (Call *)self;
  if (PyObject_SetAttr(function, s_direct, self) < 0) return nullptr;
  Py_XINCREF(f->func_code);
  Py_XSETREF(c->body, f->func_code);
  Py_XINCREF(f->func_defaults);
  Py_XSETREF(c->defaults, f->func_defaults);
  if (f->vectorcall != function_call) {
    g_interpret = f->vectorcall;
#if PY_VERSION_HEX >= 0x030c0000
    PyFunction_SetVectorcall(f, function_call);
#else
    f->vectorcall = function_call;
#endif
  }
  Py_RETURN_NONE;
}

int call_init(PyObject *self, PyObject *args, PyObject *) {
  Call *c = (Call *)self;
  const char *name;
  PyObject *function, *globals, *tensor;
  if (!PyArg_ParseTuple(args, "sOO!O!", &name, &function, &PyDict_Type, &globals, &PyType_Type, &tensor)) return -1;
  int kind = 0;
  while (kind < KINDS && std::strcmp(kShapes[kind].name, name)) ++kind;
  if (kind == KINDS) {
    PyErr_SetString(PyExc_ValueError, name);
    return -1;
  }
  c->kind = kind;
  c->vectorcall = call;
  Py_INCREF(function);
  Py_XSETREF(c->function, function);
  Py_INCREF(globals);
  Py_XSETREF(c->globals, globals);
  Py_INCREF(tensor);
  Py_XSETREF(c->tensor, (PyTypeObject *)tensor);
  return 0;
}
int call_traverse(PyObject *self, visitproc visit, void *arg) {
  Call *c = (Call *)self;
  Py_VISIT(c->function);
  Py_VISIT(c->globals);
  Py_VISIT(c->tensor);
  Py_VISIT(c->body);
  Py_VISIT(c->defaults);
  return 0;
}
int call_clear(PyObject *self) {
  Call *c = (Call *)self;
  c->address = nullptr;
  Py_CLEAR(c->function);
  Py_CLEAR(c->globals);
  Py_CLEAR(c->tensor);
  Py_CLEAR(c->body);
  Py_CLEAR(c->defaults);
  return 0;
}
void call_dealloc(PyObject *self) {
  PyObject_GC_UnTrack(self);
  call_clear(self);
  Py_TYPE(self)->tp_free(self);
}
PyObject *call_get_address(PyObject *self, void *) { return PyLong_FromVoidPtr(((Call *)self)->address); }
int call_set_address(PyObject *self, PyObject *value, void *) {
  void *p = value ? PyLong_AsVoidPtr(value) : nullptr;
  if (PyErr_Occurred()) return -1;
  ((Call *)self)->address = p;
  return 0;
}
PyGetSetDef call_getset[] = {{"address", call_get_address, call_set_address, nullptr, nullptr}, {nullptr}};
PyMethodDef call_methods[] = {{"serve", call_serve, METH_O, "Calls of a function go this way first."}, {nullptr}};

PyMethodDef module_methods[] = {{"describe", (PyCFunction)(void (*)())module_describe, METH_FASTCALL, "The descriptor of a Tensor's fields, or None."}, {nullptr}};
PyModuleDef module_def = {PyModuleDef_HEAD_INIT, "_call", nullptr, -1, module_methods};

}  // namespace

PyMODINIT_FUNC PyInit__call() {
  DescType.tp_basicsize = sizeof(Desc);
  DescType.tp_flags = Py_TPFLAGS_DEFAULT;
  DescType.tp_new = PyType_GenericNew;
  DescType.tp_as_buffer = &desc_as_buffer;
  CallType.tp_basicsize = sizeof(Call);
  CallType.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_GC | Py_TPFLAGS_HAVE_VECTORCALL;
  CallType.tp_vectorcall_offset = offsetof(Call, vectorcall);
  CallType.tp_call = PyVectorcall_Call;
  CallType.tp_new = PyType_GenericNew;
  CallType.tp_init = call_init;
  CallType.tp_traverse = call_traverse;
  CallType.tp_clear = call_clear;
  CallType.tp_dealloc = call_dealloc;
  CallType.tp_getset = call_getset;
  CallType.tp_methods = call_methods;
  if (PyType_Ready(&DescType) < 0 || PyType_Ready(&CallType) < 0) return nullptr;
  for (int k = 0; k < KINDS; ++k)
    for (int i = 0; i < kShapes[k].total; ++i)
      if (!g_params[k][i] && !(g_params[k][i] = PyUnicode_InternFromString(kShapes[k].params[i]))) return nullptr;
  struct { PyObject **s; const char *text; } names[] = {{&s_direct, "_direct"}, {&s_desc, "_desc"}, {&s_raw_stream, "_raw_stream"}, {&s_data_ptr, "data_ptr"}, {&s_numel, "numel"},
                                                        {&s_check, "_check"}, {&s_unary, "UNARY_CODE"}, {&s_binary, "BINARY_CODE"}, {&s_reduce, "REDUCE_CODE"},
                                                        {&s_dtype, "DTYPE_CODE"}, {&s_ref, "_ref"}, {&s_base, "base"}, {&s_dtype_field, "dtype"}, {&s_sizes, "sizes"},
                                                        {&s_strides, "strides"}, {&s_offset, "offset"}, {&s_device, "device"}, {&s_byteswapped, "byteswapped"}};
  for (auto &e : names)
    if (!*e.s && !(*e.s = PyUnicode_InternFromString(e.text))) return nullptr;
  PyObject *m = PyModule_Create(&module_def);
  if (!m) return nullptr;
  if (PyModule_AddIntConstant(m, "INTERFACE", kInterface) < 0) return nullptr;
  Py_INCREF(&DescType);
  Py_INCREF(&CallType);
  if (PyModule_AddObject(m, "Desc", (PyObject *)&DescType) < 0 || PyModule_AddObject(m, "Call", (PyObject *)&CallType) < 0) return nullptr;
  return m;
}
