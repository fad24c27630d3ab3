// Argument marshalling of the binding's per-call path, native: from the tensors a caller passes to one call of the C ABI.
//
// Every function takes the address of an entry point (of the library that is loaded), then the arguments of the Python
// function of the same name, and returns the entry's status -- or None where the call is not of the plain form: anything but
// exact torch tensors in device memory, of the types, layouts and sizes that the checks of the Python functions ask for.  Those
// then run, and convert or refuse as ever, so no check and no error message lives here.  No result and no address is kept
// from one call to the next.
//
// Why: at a few images a block's kernels take less time than enqueuing them, and ctypes with attribute lookups on some
// ten tensors took 2.6 us of masker_ex's 10 and 5 us of the packed block's 17.
#include <torch/csrc/autograd/python_variable.h>

#include "lasnet.h"

namespace {

PyObject *g_current_device, *g_current_stream;       // torch._C._cuda_getDevice, _cuda_getCurrentRawStream

// a tensor that is no subclass (those may override what is read here), or nullptr
inline const at::Tensor* tensor(PyObject* o) { return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr; }

struct Plain {                                       // false from any of these: not the plain form
  bool ok = true;
  bool need(bool v) { return ok = ok && v; }

  bool map(PyObject* o, lasnet_tensor& d) {          // a feature map
    const at::Tensor* t = tensor(o);
    if (!need(t && t->defined() && t->dim() == 4 && t->is_cuda() && t->is_contiguous())) return false;
    const auto ty = t->scalar_type();
    if (!need(ty == at::kFloat || ty == at::kBFloat16)) return false;
    int32_t* sizes[4] = {&d.n, &d.h, &d.w, &d.c};
    for (int i = 0; i < 4; ++i) {
      if (!need(t->size(i) <= INT32_MAX)) return false;
      *sizes[i] = (int32_t)t->size(i);
    }
    d.data = t->data_ptr();
    d.dtype = ty == at::kFloat ? LASNET_F32 : LASNET_BF16;
    return true;
  }
  template <class T>
  T* of_type(PyObject* o, at::ScalarType ty) {
    const at::Tensor* t = tensor(o);
    if (!need(t && t->defined() && t->scalar_type() == ty && t->is_cuda() && t->is_contiguous())) return nullptr;
    return (T*)t->data_ptr();
  }
  const float* bias(PyObject* o, int64_t n) {
    const float* p = of_type<const float>(o, at::kFloat);
    return ok && need(tensor(o)->numel() == n) ? p : nullptr;
  }
  template <class T>
  T* any(PyObject* o) {                              // what the Python function passes on unchecked
    const at::Tensor* t = tensor(o);
    return need(t && t->defined()) ? (T*)t->data_ptr() : nullptr;
  }
  const void* weight(PyObject* o, const lasnet_tensor& x, std::initializer_list<int64_t> shape) {
    const at::Tensor* t = tensor(o);
    const auto ty = x.dtype == LASNET_F32 ? at::kFloat : at::kBFloat16;
    if (!need(t && t->defined() && t->scalar_type() == ty && t->is_cuda() && t->is_contiguous() && t->sizes() == at::IntArrayRef(shape))) return nullptr;
    return t->data_ptr();
  }
  int integer(PyObject* o) {
    if (!need(PyLong_CheckExact(o))) return 0;
    int over = 0;
    const long v = PyLong_AsLongAndOverflow(o, &over);
    need(!over && v >= INT32_MIN && v <= INT32_MAX);
    return (int)v;
  }
  float real(PyObject* o) {
    if (PyFloat_CheckExact(o)) return (float)PyFloat_AS_DOUBLE(o);
    return (float)integer(o);
  }
  // the list: storage for every cell of the map (the kernels may read entries past the count)
  void list(PyObject* idx, PyObject* count, const lasnet_tensor& x, int S, const int32_t*& i, const int32_t*& c) {
    i = c = nullptr;
    if (count != Py_None) c = of_type<const int32_t>(count, at::kInt);
    if (idx != Py_None) {
      i = of_type<const int32_t>(idx, at::kInt);
      if (ok) need(S > 0 && x.h % S == 0 && x.w % S == 0 && tensor(idx)->numel() >= (int64_t)x.n * (x.h / S) * (x.w / S));
    }
  }
};

void* current_stream() {
  PyObject* device = PyObject_CallNoArgs(g_current_device);
  if (!device) return nullptr;
  PyObject* stream = PyObject_CallOneArg(g_current_stream, device);
  Py_DECREF(device);
  if (!stream) return nullptr;
  void* st = PyLong_AsVoidPtr(stream);
  Py_DECREF(stream);
  return st;
}

// body(plain) marshals and, where plain.ok, calls the entry
template <class Body>
PyObject* call(Py_ssize_t n, Py_ssize_t want, Body&& body) {
  if (n != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  int status = 0;
  Plain p;
  try {
    status = body(p);
  } catch (const std::exception&) {                  // a tensor without storage, for instance
    p.ok = false;
  }
  if (PyErr_Occurred()) return nullptr;
  if (!p.ok) Py_RETURN_NONE;
  return PyLong_FromLong(status);
}
template <class F>
F* entry(PyObject* address) { return (F*)PyLong_AsVoidPtr(address); }

#define ENQUEUE(...)              \
  void* st = current_stream();    \
  if (PyErr_Occurred()) return 0; \
  int status;                     \
  Py_BEGIN_ALLOW_THREADS          \
  status = __VA_ARGS__;           \
  Py_END_ALLOW_THREADS            \
  return status

// (x, Wm, bm, S, thr, mask, idx, count, pass_out)
PyObject* masker_ex(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 10, [&](Plain& p) {
    lasnet_tensor x, o;
    p.map(a[1], x);
    const float* Wm = p.of_type<const float>(a[2], at::kFloat);
    const float bm = p.real(a[3]), thr = p.real(a[5]);
    const int S = p.integer(a[4]);
    uint8_t* mask = p.any<uint8_t>(a[6]);
    int32_t *idx = p.any<int32_t>(a[7]), *count = p.any<int32_t>(a[8]);
    if (a[9] != Py_None) p.map(a[9], o);
    if (!p.ok || !p.need(S > 0 && x.h % S == 0 && x.w % S == 0)) return 0;
    lasnet_tensor* out = a[9] != Py_None ? &o : nullptr;
    auto* f = entry<decltype(lasnet_masker_ex)>(a[0]);
    ENQUEUE(f(&x, Wm, bm, S, thr, mask, idx, count, out, st));
  });
}

// (x, idx, count, S, M, packed, need, b1, b2, b3, out, flags); need: bytes that `packed` must hold, 0 if the shape has none
PyObject* block_packed(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 13, [&](Plain& p) {
    lasnet_tensor x, o;
    p.map(a[1], x);
    const int S = p.integer(a[4]), M = p.integer(a[5]), flags = p.integer(a[12]);
    const int32_t *idx, *count;
    p.list(a[2], a[3], x, S, idx, count);
    const void* packed = p.any<const void>(a[6]);
    if (!p.ok) return 0;
    const size_t need = entry<decltype(lasnet_packed_weights_bytes)>(a[7])(LASNET_BF16, x.c, M, S);
    p.need((size_t)tensor(a[6])->nbytes() >= need);
    const float *b1 = p.bias(a[8], M), *b2 = p.bias(a[9], M), *b3 = p.bias(a[10], x.c);
    p.map(a[11], o);
    if (!p.ok) return 0;
    auto* f = entry<decltype(lasnet_sparse_bottleneck_packed)>(a[0]);
    ENQUEUE(f(&x, idx, count, S, M, packed, b1, b2, b3, &o, (uint32_t)flags, st));
  });
}

// (x, idx, count, mask, S, M, packed, b1, b2, b3, out, workspace, flags)
PyObject* block_planned(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 14, [&](Plain& p) {
    lasnet_tensor x, o;
    p.map(a[1], x);
    const int S = p.integer(a[5]), M = p.integer(a[6]), flags = p.integer(a[13]);
    const int32_t *idx, *count;
    p.list(a[2], a[3], x, S, idx, count);
    const uint8_t* mask = a[4] == Py_None ? nullptr : p.of_type<const uint8_t>(a[4], at::kByte);
    const void* packed = p.any<const void>(a[7]);
    if (!p.ok) return 0;
    const float *b1 = p.bias(a[8], M), *b2 = p.bias(a[9], M), *b3 = p.bias(a[10], x.c);
    p.map(a[11], o);
    void* workspace = a[12] == Py_None ? nullptr : p.any<void>(a[12]);
    if (!p.ok) return 0;
    const size_t bytes = a[12] == Py_None ? 0 : tensor(a[12])->nbytes();
    auto* f = entry<decltype(lasnet_sparse_bottleneck_planned)>(a[0]);
    ENQUEUE(f(&x, idx, count, mask, S, M, packed, b1, b2, b3, &o, (uint32_t)flags, workspace, bytes, st));
  });
}

struct Weights { const void *W1, *W2, *W3; const float *b1, *b2, *b3; int M; };
// w: W1, b1, W2, b2, W3, b3
inline void weights(Plain& p, PyObject* const* w, const lasnet_tensor& x, Weights& r) {
  const at::Tensor* W1 = tensor(w[0]);
  if (!p.need(W1 && W1->defined() && W1->dim() == 2 && W1->size(0) <= INT32_MAX)) return;
  const int64_t M = W1->size(0);
  r.M = (int)M;
  r.W1 = p.weight(w[0], x, {M, x.c});
  r.b1 = p.bias(w[1], M);
  r.W2 = p.weight(w[2], x, {M, 3, 3, M});
  r.b2 = p.bias(w[3], M);
  r.W3 = p.weight(w[4], x, {x.c, M});
  r.b3 = p.bias(w[5], x.c);
}

// (x, idx, count, S, W1, b1, W2, b2, W3, b3, out, flags)
PyObject* block_ex(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 13, [&](Plain& p) {
    lasnet_tensor x, o;
    if (!p.map(a[1], x)) return 0;
    const int S = p.integer(a[4]), flags = p.integer(a[12]);
    const int32_t *idx, *count;
    p.list(a[2], a[3], x, S, idx, count);
    Weights w;
    weights(p, a + 5, x, w);
    p.map(a[11], o);
    if (!p.ok) return 0;
    auto* f = entry<decltype(lasnet_sparse_bottleneck_ex)>(a[0]);
    ENQUEUE(f(&x, idx, count, S, w.M, w.W1, w.b1, w.W2, w.b2, w.W3, w.b3, &o, (uint32_t)flags, st));
  });
}

// (x, W1, b1, W2, b2, W3, b3, out, flags)
PyObject* block_dense(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return call(n, 10, [&](Plain& p) {
    lasnet_tensor x, o;
    if (!p.map(a[1], x)) return 0;
    const int flags = p.integer(a[9]);
    Weights w;
    weights(p, a + 2, x, w);
    p.map(a[8], o);
    if (!p.ok) return 0;
    auto* f = entry<decltype(lasnet_dense_bottleneck)>(a[0]);
    ENQUEUE(f(&x, w.M, w.W1, w.b1, w.W2, w.b2, w.W3, w.b3, &o, (uint32_t)flags, st));
  });
}

PyMethodDef methods[] = {
    {"masker_ex", (PyCFunction)(void*)masker_ex, METH_FASTCALL, nullptr},
    {"block_packed", (PyCFunction)(void*)block_packed, METH_FASTCALL, nullptr},
    {"block_planned", (PyCFunction)(void*)block_planned, METH_FASTCALL, nullptr},
    {"block_ex", (PyCFunction)(void*)block_ex, METH_FASTCALL, nullptr},
    {"block_dense", (PyCFunction)(void*)block_dense, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* torch = PyImport_ImportModule("torch._C");
  if (!torch) return nullptr;
  g_current_device = PyObject_GetAttrString(torch, "_cuda_getDevice");
  g_current_stream = PyObject_GetAttrString(torch, "_cuda_getCurrentRawStream");
  Py_DECREF(torch);
  if (!g_current_device || !g_current_stream) return nullptr;
  return PyModule_Create(&module);
}
