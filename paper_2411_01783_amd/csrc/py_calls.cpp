// The calls of binding.py that a serving loop makes for every step, as a CPython module: the
// arguments are read from the tensors, results and workspaces allocated and the C ABI called
// without going through Python objects for each of them. Marshalling a small call in Python
// (ctypes, torch.empty, torch.cuda.current_stream) took 6 to 13 us, two to four times as long
// as issuing its kernels; here it is about 1 us.
//
// The library itself is loaded by binding.py, which hands over the addresses of its functions.
#include <Python.h>

#include <ATen/ATen.h>
#include <torch/csrc/Dtype.h>
#include <torch/csrc/autograd/python_variable.h>

#include "cp_attn.h"

namespace {

struct Functions {
  decltype(&cp_workspace_bytes) workspace_bytes;
  decltype(&cp_attn_partial) partial;
  decltype(&cp_attn_decode) decode;
  decltype(&cp_attn_decode_static) decode_static;
  decltype(&cp_attn_merge) merge;
  decltype(&cp_kv_append) append;
  decltype(&cp_ring_passkv) ring[3];  // pass-KV, pass-Q, pass-Q decode
} fn = {};

PyObject* get_device = nullptr;      // torch._C._cuda_getDevice
PyObject* get_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream

struct Raised {};  // a Python error is set

[[noreturn]] void raise(PyObject* type, const char* what) {
  PyErr_SetString(type, what);
  throw Raised{};
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a torch tensor");
  return THPVariable_Unpack(o);
}
void* pointer(const at::Tensor& t) {
  if (!t.is_contiguous())
    raise(PyExc_AssertionError, "tensors handed to the C ABI must be contiguous");
  return const_cast<void*>(t.const_data_ptr());
}
void* pointer(PyObject* o) { return o == Py_None ? nullptr : pointer(tensor(o)); }

int32_t dtype_code(at::ScalarType t) {
  if (t == at::kBFloat16) return CP_BF16;
  if (t == at::kFloat) return CP_FP32;
  PyErr_Format(PyExc_TypeError, "unsupported dtype %s", at::toString(t));
  throw Raised{};
}
at::ScalarType dtype_or(PyObject* o, at::ScalarType other) {
  if (o == Py_None) return other;
  if (!THPDtype_Check(o)) raise(PyExc_TypeError, "out_dtype must be a torch dtype");
  return reinterpret_cast<THPDtype*>(o)->scalar_type;
}
float number(PyObject* o) {
  const double x = PyFloat_AsDouble(o);
  if (x == -1.0 && PyErr_Occurred()) throw Raised{};
  return (float)x;
}

// A raw stream given as a number, or torch's current one.
void* stream_of(PyObject* o) {
  if (o != Py_None) {
    void* const s = PyLong_AsVoidPtr(o);
    if (s == nullptr && PyErr_Occurred()) throw Raised{};
    return s;
  }
  PyObject* const dev = PyObject_CallNoArgs(get_device);
  if (dev == nullptr) throw Raised{};
  PyObject* const raw = PyObject_CallOneArg(get_raw_stream, dev);
  Py_DECREF(dev);
  if (raw == nullptr) throw Raised{};
  void* const s = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  if (s == nullptr && PyErr_Occurred()) throw Raised{};
  return s;
}

struct Workspace {
  at::Tensor own;
  void* ptr = nullptr;
  size_t bytes = 0;
  void set(const at::Tensor& t) {
    const uintptr_t p = (uintptr_t)t.const_data_ptr(), a = (p + 255) & ~(uintptr_t)255;
    ptr = (void*)a;
    bytes = (size_t)(t.numel() - (int64_t)(a - p));
  }
};
void use_workspace(Workspace& w, PyObject* given, const cp_shape& s, int32_t kind,
                   const at::Tensor& like) {
  if (given != Py_None) {
    w.set(tensor(given));
    return;
  }
  const size_t need = fn.workspace_bytes(&s, kind);
  if (need == 0) return;
  w.own = at::empty({(int64_t)need + 256}, like.options().dtype(at::kByte));
  w.set(w.own);
}

cp_shape rows_shape(const at::Tensor& q, const at::Tensor& k, int64_t batch, float scale,
                    int32_t flags) {
  if (q.dim() != 3 || k.dim() != 3) raise(PyExc_ValueError, "q and k must have three dimensions");
  cp_shape s = {};
  s.dtype = dtype_code(q.scalar_type());
  s.head_dim = (int32_t)q.size(2);
  s.n_q_heads = (int32_t)q.size(1);
  s.n_kv_heads = (int32_t)k.size(1);
  s.batch = (int32_t)batch;
  s.flags = flags;
  s.total_q = q.size(0);
  s.total_kv = k.size(0);
  s.softmax_scale = scale;
  return s;
}

// `given`, or a new tensor.
at::Tensor result(PyObject* given, at::IntArrayRef sizes, const at::Tensor& like,
                  at::ScalarType dtype) {
  return given != Py_None ? tensor(given) : at::empty(sizes, like.options().dtype(dtype));
}
PyObject* object(PyObject* given, const at::Tensor& t) {
  if (given == Py_None) return THPVariable_Wrap(t);
  Py_INCREF(given);
  return given;
}
PyObject* pair(PyObject* a, PyObject* b) {
  if (a == nullptr || b == nullptr) {
    Py_XDECREF(a);
    Py_XDECREF(b);
    return nullptr;
  }
  PyObject* const t = PyTuple_Pack(2, a, b);
  Py_DECREF(a);
  Py_DECREF(b);
  return t;
}
PyObject* status(int rc) { return PyLong_FromLong(rc); }

// Other threads run while the library is called, as they do in a ctypes call: a launch blocks
// once the stream's queue is full. The tensors are the caller's arguments or held on the stack.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F, typename... A>
int call(F f, A... args) {
  const Unlocked u;
  return f(args...);
}

void arguments(Py_ssize_t n, Py_ssize_t want) {
  if (n != want) raise(PyExc_TypeError, "wrong number of arguments");
  if (fn.decode == nullptr) raise(PyExc_RuntimeError, "the library is not loaded");
}

// Every function returns its result, or the (nonzero) status of the C call as a number.
template <typename F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (const Raised&) {
    return nullptr;
  } catch (const std::exception& e) {   // of torch: out of memory, no device
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// q, k, v, q_pos, kv_pos, cu_seqlens_q, cu_seqlens_kv, out_dtype, scale, out, lse, workspace, stream
PyObject* partial(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    arguments(n, 13);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
    const int64_t batch = a[5] == Py_None ? 1 : tensor(a[5]).numel() - 1;
    const cp_shape s = rows_shape(q, k, batch, number(a[8]), 0);
    const at::Tensor out = result(a[9], q.sizes(), q, dtype_or(a[7], q.scalar_type()));
    const at::Tensor lse = result(a[10], {q.size(0), q.size(1)}, q, at::kFloat);
    Workspace w;
    use_workspace(w, a[11], s, CP_WS_PARTIAL, q);
    const int rc = call(fn.partial, &s, pointer(q), pointer(k), pointer(a[2]), (int32_t*)pointer(a[3]),
                              (int32_t*)pointer(a[4]), (int32_t*)pointer(a[5]),
                              (int32_t*)pointer(a[6]), pointer(out), (float*)pointer(lse),
                              dtype_code(out.scalar_type()), w.ptr, w.bytes, stream_of(a[12]));
    return rc != CP_OK ? status(rc) : pair(object(a[9], out), object(a[10], lse));
  });
}

// q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out_dtype, scale, out, lse, workspace, stream, unique
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    arguments(n, 14);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]);
    const int unique = PyObject_IsTrue(a[13]);
    if (unique < 0) throw Raised{};
    const cp_shape s = rows_shape(q, k, tensor(a[5]).numel() - 1, number(a[8]),
                                  unique ? CP_SHAPE_UNIQUE_BID : 0);
    const at::Tensor out = result(a[9], q.sizes(), q, dtype_or(a[7], q.scalar_type()));
    const at::Tensor lse = result(a[10], {q.size(0), q.size(1)}, q, at::kFloat);
    Workspace w;
    use_workspace(w, a[11], s, CP_WS_DECODE, q);
    const int rc = call(fn.decode, &s, pointer(q), pointer(k), pointer(a[2]), (int32_t*)pointer(a[3]),
                             (int32_t*)pointer(a[4]), (int32_t*)pointer(a[5]),
                             (int32_t*)pointer(a[6]), pointer(out), (float*)pointer(lse),
                             dtype_code(out.scalar_type()), w.ptr, w.bytes, stream_of(a[12]));
    return rc != CP_OK ? status(rc) : pair(object(a[9], out), object(a[10], lse));
  });
}

// q, k, v, q_pos, kv_pos, cu_seqlens_kv, bid, out, lse, scale, stream, unique
PyObject* decode_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    arguments(n, 12);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &out = tensor(a[7]);
    const int unique = PyObject_IsTrue(a[11]);
    if (unique < 0) throw Raised{};
    const cp_shape s = rows_shape(q, k, tensor(a[5]).numel() - 1, number(a[9]),
                                  unique ? CP_SHAPE_UNIQUE_BID : 0);
    return status(call(fn.decode_static, &s, pointer(q), pointer(k), pointer(a[2]),
                                   (int32_t*)pointer(a[3]), (int32_t*)pointer(a[4]),
                                   (int32_t*)pointer(a[5]), (int32_t*)pointer(a[6]), pointer(out),
                                   (float*)pointer(a[8]), dtype_code(out.scalar_type()),
                                   stream_of(a[10])));
  });
}

// outs, lses (sequences), out_dtype, out, lse_out, want_lse, stream
PyObject* merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
  PyObject *outs = nullptr, *lses = nullptr;
  PyObject* const r = guarded([&]() -> PyObject* {
    arguments(n, 7);
    outs = PySequence_Fast(a[0], "outs must be a sequence of tensors");
    if (outs == nullptr) throw Raised{};
    lses = PySequence_Fast(a[1], "lses must be a sequence of tensors");
    if (lses == nullptr) throw Raised{};
    const Py_ssize_t parts = PySequence_Fast_GET_SIZE(outs);
    if (parts == 0) raise(PyExc_IndexError, "list index out of range");
    if (PySequence_Fast_GET_SIZE(lses) != parts)
      raise(PyExc_IndexError, "outs and lses differ in length");
    const at::Tensor& o0 = tensor(PySequence_Fast_GET_ITEM(outs, 0));
    if (o0.dim() < 1) raise(PyExc_IndexError, "partial outputs need a channel dimension");
    const int64_t d = o0.size(-1), rows = d > 0 ? o0.numel() / d : 0;
    const at::Tensor out = result(a[3], o0.sizes(), o0, dtype_or(a[2], o0.scalar_type()));
    const int want = PyObject_IsTrue(a[5]);
    if (want < 0) throw Raised{};
    at::Tensor lse;
    if (a[4] != Py_None) lse = tensor(a[4]);
    else if (want) lse = at::empty(o0.sizes().slice(0, o0.dim() - 1), o0.options().dtype(at::kFloat));
    // (the C call rejects more than CP_MAX_PARTS before it reads the arrays)
    const void* op[CP_MAX_PARTS];
    const float* lp[CP_MAX_PARTS];
    for (Py_ssize_t i = 0; i < parts && i < CP_MAX_PARTS; ++i) {
      op[i] = pointer(PySequence_Fast_GET_ITEM(outs, i));
      lp[i] = (const float*)pointer(PySequence_Fast_GET_ITEM(lses, i));
    }
    const int rc = call(fn.merge, rows, (int32_t)d, (int32_t)parts, op, lp,
                            dtype_code(o0.scalar_type()), pointer(out),
                            dtype_code(out.scalar_type()),
                            lse.defined() ? (float*)pointer(lse) : nullptr, stream_of(a[6]));
    if (rc != CP_OK) return status(rc);
    PyObject* l;
    if (lse.defined()) {
      l = object(a[4], lse);
    } else {
      l = Py_None;
      Py_INCREF(l);
    }
    return pair(object(a[3], out), l);
  });
  Py_XDECREF(outs);
  Py_XDECREF(lses);
  return r;
}

// k_new, v_new, pos_new, cu_seqlens_new, k, v, kv_pos, cu, used, dropped (of the cache), slots,
// batch, stream
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    arguments(n, 13);
    const at::Tensor &k = tensor(a[0]), &cache = tensor(a[4]);
    const int64_t slots = PyLong_AsLongLong(a[10]), batch = PyLong_AsLongLong(a[11]);
    if (PyErr_Occurred()) throw Raised{};
    if (k.dim() != 3) raise(PyExc_ValueError, "k_new must have three dimensions");
    if (k.scalar_type() != cache.scalar_type() || cache.size(1) != k.size(1) ||
        cache.size(2) != k.size(2))
      raise(PyExc_ValueError, "new K/V rows do not match the cache's row shape or dtype");
    if (tensor(a[3]).numel() != batch + 1 || tensor(a[2]).numel() != k.size(0))
      raise(PyExc_ValueError, "cu_seqlens_new / pos_new sizes do not match");
    cp_shape s = {};
    s.dtype = dtype_code(k.scalar_type());
    s.head_dim = (int32_t)k.size(2);
    s.n_q_heads = s.n_kv_heads = (int32_t)k.size(1);
    s.batch = (int32_t)batch;
    s.total_q = k.size(0);
    s.total_kv = slots;
    return status(call(fn.append, &s, pointer(k), pointer(a[1]), (int32_t*)pointer(a[2]),
                            (int32_t*)pointer(a[3]), pointer(cache), pointer(a[5]),
                            (int32_t*)pointer(a[6]), (int32_t*)pointer(a[7]),
                            (int32_t*)pointer(a[8]), (int32_t*)pointer(a[9]), stream_of(a[12])));
  });
}

// which driver, address of a cp_ring_desc, stream
PyObject* ring(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    arguments(n, 3);
    const long which = PyLong_AsLong(a[0]);
    if (which < 0 || which > 2) raise(PyExc_ValueError, "no such ring driver");
    void* const desc = PyLong_AsVoidPtr(a[1]);
    if (PyErr_Occurred()) throw Raised{};
    return status(call(fn.ring[which], (const cp_ring_desc*)desc, stream_of(a[2])));
  });
}

// addresses of cp_workspace_bytes, cp_attn_partial, cp_attn_decode, cp_attn_decode_static,
// cp_attn_merge, cp_kv_append, cp_ring_passkv, cp_ring_passq, cp_ring_passq_decode
PyObject* connect(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 9) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  void* p[9];
  for (int i = 0; i < 9; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function is missing");
      return nullptr;
    }
  }
  if (get_device == nullptr) {
    PyObject* const m = PyImport_ImportModule("torch._C");
    if (m == nullptr) return nullptr;
    get_device = PyObject_GetAttrString(m, "_cuda_getDevice");
    get_raw_stream = PyObject_GetAttrString(m, "_cuda_getCurrentRawStream");
    Py_DECREF(m);
    if (get_device == nullptr || get_raw_stream == nullptr) {
      Py_CLEAR(get_device);
      Py_CLEAR(get_raw_stream);
      return nullptr;
    }
  }
  fn.workspace_bytes = (decltype(fn.workspace_bytes))p[0];
  fn.partial = (decltype(fn.partial))p[1];
  fn.decode = (decltype(fn.decode))p[2];
  fn.decode_static = (decltype(fn.decode_static))p[3];
  fn.merge = (decltype(fn.merge))p[4];
  fn.append = (decltype(fn.append))p[5];
  for (int i = 0; i < 3; ++i) fn.ring[i] = (decltype(fn.ring[0]))p[6 + i];
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"connect", (PyCFunction)(void*)connect, METH_FASTCALL, nullptr},
    {"partial", (PyCFunction)(void*)partial, METH_FASTCALL, nullptr},
    {"decode", (PyCFunction)(void*)decode, METH_FASTCALL, nullptr},
    {"decode_static", (PyCFunction)(void*)decode_static, METH_FASTCALL, nullptr},
    {"merge", (PyCFunction)(void*)merge, METH_FASTCALL, nullptr},
    {"append", (PyCFunction)(void*)append, METH_FASTCALL, nullptr},
    {"ring", (PyCFunction)(void*)ring, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_py_calls", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__py_calls(void) { return PyModule_Create(&module); }
