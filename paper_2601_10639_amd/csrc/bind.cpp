// The hot calls of stemlib.py natively: tensors to pointers, the current stream, and the C call without the interpreter's lock.
//
// A small layer's call spends as long on the host as on the GPU: a launch takes 2.7 to 3.5 us there, and forward_residual's arguments took
// 2.9 in Python (0.22 for each tensor's checks, 0.36 for the stream, 0.6 for ctypes), 0.46 here.  A training step of 128 tokens of 64 x 256
// fp32, four calls and six launches, 33.8 -> 24.0 us.
//
// Only the ordinary call is made here: plain torch tensors of the right type in contiguous device memory, ints, floats and bools.
// Every function returns None, having done nothing, where anything else is among the arguments, and stemlib.py then makes the call as it
// does without this module: its checks say what is wrong, or take what this one does not know.  It looks into torch's and Python's objects,
// so stemlib.py uses it only with the versions it was built for.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include "../../include/stem.h"

namespace {

PyObject *g_ctx_type, *g_get_device, *g_raw_stream, *g_handle, *g_value, *g_dtype, *g_cuda_stream;   // set by setup()
bool g_off = true;                                        // before setup(), and in a forked process

struct Unusual {};

struct Hold {                  // a new reference, or Unusual
  PyObject* o;
  explicit Hold(PyObject* p) : o(p) {
    if (!p) { PyErr_Clear(); throw Unusual(); }
  }
  ~Hold() { Py_DECREF(o); }
};

enum Kind { ACT, F32, I32 };   // ACT: the context's type

// The arguments of one call
struct Args {
  PyObject* const* v;
  int dtype;
  mutable bool device_seen;    // a device tensor is among them: the runtime is up

  template <class T = void>
  T* ptr(int i, Kind kind) const {
    PyObject* const o = v[i];
    if (o == Py_None) return nullptr;
    if (!THPVariable_CheckExact(o)) throw Unusual();
    const at::Tensor& t = THPVariable_Unpack(o);
    const at::ScalarType want = kind == I32 ? at::kInt : kind == ACT && dtype == STEM_BF16 ? at::kBFloat16 : at::kFloat;
    if (t.layout() != at::kStrided || t.scalar_type() != want || !t.is_cuda() || !t.is_contiguous()) throw Unusual();
    device_seen = true;
    // (as data_ptr() in Python: a tensor that shares its storage with another until one is written gets its own first.  Inputs too, as a
    // call may write to the same tensor)
    return static_cast<T*>(t.mutable_data_ptr());
  }

  static int64_t as_integer(PyObject* o) {
    if (!PyLong_CheckExact(o)) throw Unusual();
    int overflow = 0;
    const int64_t x = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow) throw Unusual();
    return x;
  }
  int64_t integer(int i) const { return as_integer(v[i]); }
  int flag(int i) const {
    if (!PyBool_Check(v[i])) throw Unusual();
    return v[i] == Py_True;
  }
  float number(int i) const {
    if (!PyFloat_CheckExact(v[i])) throw Unusual();
    return (float)PyFloat_AS_DOUBLE(v[i]);
  }
  void* pointer(int i) const { return v[i] == Py_None ? nullptr : reinterpret_cast<void*>(integer(i)); }

  // argument i, or where it is None the rows of tensor t (0 where that is None and may be)
  int64_t rows(int i, int t, bool none_is_0 = false) const {
    if (v[i] != Py_None) return integer(i);
    if (v[t] == Py_None && none_is_0) return 0;
    if (!THPVariable_CheckExact(v[t])) throw Unusual();
    const at::Tensor& x = THPVariable_Unpack(v[t]);
    if (x.dim() < 1) throw Unusual();
    return x.size(0);
  }

  // a stream's handle, or the current stream's; after the tensors
  void* stream(int i) const {
    if (PyLong_CheckExact(v[i])) return reinterpret_cast<void*>(integer(i));
    if (v[i] != Py_None) return reinterpret_cast<void*>(as_integer(Hold(PyObject_GetAttr(v[i], g_cuda_stream)).o));
    if (!device_seen) throw Unusual();
    const Hold device(PyObject_CallNoArgs(g_get_device));
    return reinterpret_cast<void*>(as_integer(Hold(PyObject_CallOneArg(g_raw_stream, device.o)).o));
  }
};

// f gets the arguments behind the context, and its handle, and returns the call.
template <class F>
PyObject* enter(PyObject* const* args, Py_ssize_t n, Py_ssize_t want, F f) {
  if (n != want + 1) return PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want + 1, n);
  if (g_off || reinterpret_cast<PyObject*>(Py_TYPE(args[0])) != g_ctx_type) Py_RETURN_NONE;
  try {
    const Hold handle(PyObject_GetAttr(args[0], g_handle)), value(PyObject_GetAttr(handle.o, g_value)), dtype(PyObject_GetAttr(args[0], g_dtype));
    stem_ctx* const c = reinterpret_cast<stem_ctx*>(Args::as_integer(value.o));   // (closed: None)
    const Args a{args + 1, (int)Args::as_integer(dtype.o), false};
    auto call = f(a, c);
    stem_status st;
    Py_BEGIN_ALLOW_THREADS
    st = call();
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  } catch (...) {              // Unusual, or what a tensor without storage throws
    Py_RETURN_NONE;
  }
}

PyObject* ffn_forward(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 12, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(11, 0), E_rows = a.rows(10, 4);
    auto x = a.ptr(0, ACT); auto ids = a.ptr<int32_t>(1, I32); auto Wg = a.ptr(2, ACT); auto Wd = a.ptr(3, ACT);
    auto E = a.ptr(4, ACT); auto y = a.ptr(5, ACT); auto G = a.ptr(6, ACT); auto H = a.ptr(7, ACT);
    auto event = a.pointer(8); auto s = a.stream(9);
    return [=] { return stem_ffn_forward(c, x, ids, Wg, Wd, E, E_rows, T, y, G, H, event, s); };
  });
}

PyObject* ffn_forward_residual(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 10, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(9, 0), E_rows = a.rows(8, 4);
    auto x = a.ptr(0, ACT); auto ids = a.ptr<int32_t>(1, I32); auto Wg = a.ptr(2, ACT); auto Wd = a.ptr(3, ACT);
    auto E = a.ptr(4, ACT); auto r = a.ptr(5, ACT); auto y = a.ptr(6, ACT); auto s = a.stream(7);
    return [=] { return stem_ffn_forward_residual(c, x, ids, Wg, Wd, E, E_rows, T, r, y, s); };
  });
}

PyObject* ffn_backward(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 16, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(15, 0), E_rows = a.rows(14, 5);
    auto dy = a.ptr(0, ACT); auto x = a.ptr(1, ACT); auto ids = a.ptr<int32_t>(2, I32); auto Wg = a.ptr(3, ACT);
    auto Wd = a.ptr(4, ACT); auto E = a.ptr(5, ACT); auto G = a.ptr(6, ACT); auto H = a.ptr(7, ACT);
    auto dx = a.ptr(8, ACT); auto dWg = a.ptr<float>(9, F32); auto dWd = a.ptr<float>(10, F32);
    auto dU = a.ptr(11, ACT); const int accumulate = a.flag(12); auto s = a.stream(13);
    return [=] { return stem_ffn_backward(c, dy, x, ids, Wg, Wd, E, E_rows, G, H, T, dx, dWg, dWd, dU, accumulate, s); };
  });
}

PyObject* ffn_up_forward(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 13, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(12, 0), E_rows = a.rows(11, 5, true);
    auto x = a.ptr(0, ACT); auto ids = a.ptr<int32_t>(1, I32); auto Wg = a.ptr(2, ACT); auto Wu = a.ptr(3, ACT);
    auto Wd = a.ptr(4, ACT); auto E = a.ptr(5, ACT); auto y = a.ptr(6, ACT); auto G = a.ptr(7, ACT);
    auto Up = a.ptr(8, ACT); auto H = a.ptr(9, ACT); auto s = a.stream(10);
    return [=] { return stem_ffn_up_forward(c, x, ids, Wg, Wu, Wd, E, E_rows, T, y, G, Up, H, s); };
  });
}

PyObject* ffn_up_backward(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 19, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(18, 0), E_rows = a.rows(17, 6, true);
    auto dy = a.ptr(0, ACT); auto x = a.ptr(1, ACT); auto ids = a.ptr<int32_t>(2, I32); auto Wg = a.ptr(3, ACT);
    auto Wu = a.ptr(4, ACT); auto Wd = a.ptr(5, ACT); auto E = a.ptr(6, ACT); auto G = a.ptr(7, ACT);
    auto Up = a.ptr(8, ACT); auto H = a.ptr(9, ACT); auto dx = a.ptr(10, ACT);
    auto dWg = a.ptr<float>(11, F32); auto dWu = a.ptr<float>(12, F32); auto dWd = a.ptr<float>(13, F32);
    auto dV = a.ptr(14, ACT); const int accumulate = a.flag(15); auto s = a.stream(16);
    return [=] { return stem_ffn_up_backward(c, dy, x, ids, Wg, Wu, Wd, E, E_rows, G, Up, H, T, dx, dWg, dWu, dWd, dV, accumulate, s); };
  });
}

PyObject* embed_grad(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 10, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(9, 0);
    auto ids = a.ptr<int32_t>(0, I32); auto dU = a.ptr(1, ACT); auto sorted = a.ptr<int32_t>(2, I32);
    auto perm = a.ptr<int32_t>(3, I32); auto uniq = a.ptr<int32_t>(4, I32); auto offs = a.ptr<int32_t>(5, I32);
    auto nu = a.ptr<int32_t>(6, I32); auto dE = a.ptr<float>(7, F32); auto s = a.stream(8);
    return [=] { return stem_embed_grad(c, ids, dU, T, sorted, perm, uniq, offs, nu, dE, s); };
  });
}

PyObject* embed_grad_presorted(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 6, [](const Args& a, stem_ctx* c) {
    const int64_t T = a.rows(5, 0);
    auto dU = a.ptr(0, ACT); auto perm = a.ptr<int32_t>(1, I32); auto offs = a.ptr<int32_t>(2, I32);
    auto dE = a.ptr<float>(3, F32); auto s = a.stream(4);
    return [=] { return stem_embed_grad_presorted(c, dU, T, perm, offs, dE, s); };
  });
}

PyObject* embed_sparse_adamw(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return enter(args, n, 15, [](const Args& a, stem_ctx* c) {
    const int64_t max_rows = a.rows(14, 2);
    auto uniq = a.ptr<int32_t>(0, I32); auto nu = a.ptr<int32_t>(1, I32); auto dE = a.ptr<float>(2, F32);
    auto E = a.ptr(3, ACT); auto master = a.ptr<float>(4, F32); auto m = a.ptr<float>(5, F32); auto v = a.ptr<float>(6, F32);
    stem_adamw_hparams hp;
    hp.lr = a.number(7); hp.beta1 = a.number(8); hp.beta2 = a.number(9); hp.eps = a.number(10); hp.weight_decay = a.number(11);
    hp.step = a.integer(12);
    auto s = a.stream(13);
    return [=] { return stem_embed_sparse_adamw(c, uniq, nu, max_rows, dE, E, master, m, v, &hp, s); };
  });
}

// (StemCtx, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream)
PyObject* setup(PyObject*, PyObject* args) {
  if (!PyArg_ParseTuple(args, "OOO", &g_ctx_type, &g_get_device, &g_raw_stream)) return nullptr;
  for (PyObject* o : {g_ctx_type, g_get_device, g_raw_stream}) Py_INCREF(o);
  g_handle = PyUnicode_InternFromString("handle");
  g_value = PyUnicode_InternFromString("value");
  g_dtype = PyUnicode_InternFromString("dtype");
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!g_handle || !g_value || !g_dtype || !g_cuda_stream) return nullptr;
  g_off = false;
  Py_RETURN_NONE;
}

PyObject* off(PyObject*, PyObject*) {
  g_off = true;
  Py_RETURN_NONE;
}

#define FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(ffn_forward), FAST(ffn_forward_residual), FAST(ffn_backward), FAST(ffn_up_forward), FAST(ffn_up_backward),
                         FAST(embed_grad), FAST(embed_grad_presorted), FAST(embed_sparse_adamw),
                         {"setup", setup, METH_VARARGS, nullptr}, {"off", off, METH_NOARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bind", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

#define STR_(x) #x
#define STR(x) STR_(x)
PyMODINIT_FUNC PyInit__bind() {
  PyObject* const m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "BUILT_FOR", "torch " TORCH_VERSION ", Python " STR(PY_MAJOR_VERSION) "." STR(PY_MINOR_VERSION)) < 0) {
    Py_DECREF(m);
    return nullptr;
  }
  return m;
}
