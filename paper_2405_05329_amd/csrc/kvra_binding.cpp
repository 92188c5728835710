// The argument marshalling of the calls a program makes per chunk, in native code.  A call through ctypes spends 1.0 us on five
// tensors (three method calls each) and 0.6 us on the call itself, of 4.7 to 5.0 us in all; with two calls per chunk and a GPU
// that needs 4 us for each, that is what a short prompt waits for.  Here the same checks and conversions read the tensor
// object directly.  What is not a plain tensor, None or an int goes through the Python function that does the same
// (kvra._ptr), so that subclasses and look-alikes are treated as before.  The module is tied to the torch and the Python it is
// compiled against; kvra.py does without it where there is none for those in use.
//
// Before -> after: kvra_append_kv 4.95 -> 2.72 us, kvra_chunk_attn 4.72 -> 2.72 us (2.5 of them in the runtime).
#define PY_SSIZE_T_CLEAN
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <exception>

#include "kvra.h"

namespace {

PyObject* g_ptr_fallback = nullptr;   // kvra._ptr
PyObject* g_cuda_stream = nullptr;    // "cuda_stream"

// The library's entry points, as bound by the importing module (one library, loaded once).
struct Entry {
  decltype(&kvra_append_kv) append_kv;
  decltype(&kvra_chunk_attn) chunk_attn;
  decltype(&kvra_rms_norm) rms_norm;
  decltype(&kvra_linear) linear;
  decltype(&kvra_qkv_proj) qkv_proj;
  decltype(&kvra_layer_chunk) layer_chunk;
} g_entry = {};

// One call's arguments, in order; the first failure sticks and leaves a Python exception set.
class Reader {
 public:
  Reader(PyObject* const* args, Py_ssize_t n, Py_ssize_t want) : args_(args) {
    if (n != want) {
      PyErr_Format(PyExc_TypeError, "%zd arguments expected, %zd given", want, n);
      ok_ = false;
    }
    if (ok_ && g_ptr_fallback == nullptr) {
      PyErr_SetString(PyExc_RuntimeError, "the binding has not been given its entry points");
      ok_ = false;
    }
  }
  bool ok() const { return ok_; }

  void* pointer() {
    if (!ok_) return nullptr;
    PyObject* const o = args_[at_++];
    if (o == Py_None) return nullptr;
    if (PyLong_Check(o)) return as_pointer(o);
    if (THPVariable_CheckExact(o)) {
      try {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_contiguous()) return fail(PyExc_ValueError, "tensor must be contiguous");
        if (!t.is_cuda()) return fail(PyExc_ValueError, "tensor must live in GPU memory");
        return t.data_ptr();
      } catch (const std::exception& e) {   // (a tensor without storage)
        return fail(PyExc_RuntimeError, e.what());
      }
    }
    PyObject* const address = PyObject_CallOneArg(g_ptr_fallback, o);
    if (address == nullptr) return fail();
    void* const p = address == Py_None ? nullptr : as_pointer(address);
    Py_DECREF(address);
    return p;
  }
  int64_t integer() {   // int(x), cut to 64 bits
    if (!ok_) return 0;
    PyObject* const o = args_[at_++];
    if (PyLong_CheckExact(o)) return mask(o);
    PyObject* const v = PyNumber_Long(o);
    if (v == nullptr) return fail(), 0;
    const int64_t r = mask(v);
    Py_DECREF(v);
    return r;
  }
  int small() { return static_cast<int>(integer()); }
  float real() {        // float(x)
    if (!ok_) return 0.0f;
    PyObject* const o = args_[at_++];
    if (PyFloat_CheckExact(o)) return static_cast<float>(PyFloat_AS_DOUBLE(o));
    PyObject* const v = PyNumber_Float(o);
    if (v == nullptr) return fail(), 0.0f;
    const float r = static_cast<float>(PyFloat_AS_DOUBLE(v));
    Py_DECREF(v);
    return r;
  }
  void* stream() {      // None, an address, or an object with one (torch.cuda.Stream)
    if (!ok_) return nullptr;
    PyObject* const o = args_[at_++];
    if (o == Py_None) return nullptr;
    if (PyLong_Check(o)) return as_pointer(o);
    PyObject* const v = PyObject_GetAttr(o, g_cuda_stream);
    if (v == nullptr) return fail();
    void* const p = v == Py_None ? nullptr : as_pointer(v);
    Py_DECREF(v);
    return p;
  }

 private:
  void* fail() {
    ok_ = false;
    return nullptr;
  }
  void* fail(PyObject* type, const char* what) {
    PyErr_SetString(type, what);
    return fail();
  }
  int64_t mask(PyObject* v) {
    const unsigned long long r = PyLong_AsUnsignedLongLongMask(v);
    if (r == static_cast<unsigned long long>(-1) && PyErr_Occurred() != nullptr) ok_ = false;
    return static_cast<int64_t>(r);
  }
  void* as_pointer(PyObject* v) {
    if (!PyLong_Check(v)) return fail(PyExc_TypeError, "an address is expected");
    return reinterpret_cast<void*>(static_cast<uintptr_t>(mask(v)));
  }
  PyObject* const* args_;
  Py_ssize_t at_ = 0;
  bool ok_ = true;
};

template <class F>
PyObject* call(const Reader& r, F&& f) {
  if (!r.ok()) return nullptr;
  int rc = 0;
  Py_BEGIN_ALLOW_THREADS   // as ctypes does: a launch may wait for room in a queue
  rc = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

PyObject* append_kv(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 13);
  void *k = r.pointer(), *v = r.pointer(), *q = r.pointer(), *kc = r.pointer(), *vc = r.pointer();
  const int64_t prefix = r.integer(), chunk = r.integer(), capacity = r.integer();
  const int H = r.small(), Hkv = r.small(), d = r.small();
  const float base = r.real();
  void* const st = r.stream();
  return call(r, [&] { return g_entry.append_kv(k, v, q, kc, vc, prefix, chunk, capacity, H, Hkv, d, base, st); });
}

PyObject* chunk_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 11);
  void *q = r.pointer(), *kc = r.pointer(), *vc = r.pointer();
  const int64_t prefix = r.integer(), chunk = r.integer();
  const int H = r.small(), Hkv = r.small(), d = r.small();
  const float scale = r.real();
  void *out = r.pointer(), *st = r.stream();
  return call(r, [&] { return g_entry.chunk_attn(q, kc, vc, prefix, chunk, H, Hkv, d, scale, out, st); });
}

PyObject* rms_norm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 7);
  void *x = r.pointer(), *gain = r.pointer(), *y = r.pointer();
  const int64_t rows = r.integer();
  const int hidden = r.small();
  const float eps = r.real();
  void* const st = r.stream();
  return call(r, [&] { return g_entry.rms_norm(x, gain, y, rows, hidden, eps, st); });
}

PyObject* linear(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 9);
  void *x = r.pointer(), *w = r.pointer(), *w2 = r.pointer(), *res = r.pointer(), *out = r.pointer();
  const int64_t m = r.integer(), cols = r.integer(), k = r.integer();
  void* const st = r.stream();
  return call(r, [&] { return g_entry.linear(x, w, w2, res, out, m, cols, k, st); });
}

PyObject* qkv_proj(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 11);
  void *x = r.pointer(), *w = r.pointer(), *q = r.pointer(), *k_out = r.pointer(), *v = r.pointer();
  const int64_t m = r.integer();
  const int H = r.small(), Hkv = r.small(), d = r.small();
  const int64_t k = r.integer();
  void* const st = r.stream();
  return call(r, [&] { return g_entry.qkv_proj(x, w, q, k_out, v, m, H, Hkv, d, k, st); });
}

PyObject* layer_chunk(PyObject*, PyObject* const* args, Py_ssize_t n) {
  Reader r(args, n, 11);
  const kvra_layer* const layer = static_cast<const kvra_layer*>(r.pointer());   // an address
  void *x = r.pointer(), *y = r.pointer(), *kc = r.pointer(), *vc = r.pointer();
  const int64_t prefix = r.integer(), chunk = r.integer(), capacity = r.integer();
  void* const ws = r.pointer();
  const int64_t bytes = r.integer();
  void* const st = r.stream();
  return call(r, [&] { return g_entry.layer_chunk(layer, x, y, kc, vc, prefix, chunk, capacity, ws, bytes, st); });
}

// bind(ptr_fallback, append_kv, chunk_attn, rms_norm, linear, qkv_proj, layer_chunk): the addresses of the entry points
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 7 || !PyCallable_Check(args[0])) {
    PyErr_SetString(PyExc_TypeError, "bind(callable, six addresses)");
    return nullptr;
  }
  void* f[6];
  for (int i = 0; i < 6; ++i) {
    f[i] = PyLong_AsVoidPtr(args[i + 1]);
    if (f[i] == nullptr) {
      if (PyErr_Occurred() == nullptr) PyErr_SetString(PyExc_ValueError, "an entry point is missing");
      return nullptr;
    }
  }
  g_entry.append_kv = reinterpret_cast<decltype(&kvra_append_kv)>(f[0]);
  g_entry.chunk_attn = reinterpret_cast<decltype(&kvra_chunk_attn)>(f[1]);
  g_entry.rms_norm = reinterpret_cast<decltype(&kvra_rms_norm)>(f[2]);
  g_entry.linear = reinterpret_cast<decltype(&kvra_linear)>(f[3]);
  g_entry.qkv_proj = reinterpret_cast<decltype(&kvra_qkv_proj)>(f[4]);
  g_entry.layer_chunk = reinterpret_cast<decltype(&kvra_layer_chunk)>(f[5]);
  Py_INCREF(args[0]);
  Py_XSETREF(g_ptr_fallback, args[0]);
  Py_RETURN_NONE;
}

#define KVRA_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {KVRA_METHOD(bind),   KVRA_METHOD(append_kv), KVRA_METHOD(chunk_attn),  KVRA_METHOD(rms_norm),
                           KVRA_METHOD(linear), KVRA_METHOD(qkv_proj),  KVRA_METHOD(layer_chunk), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_kvra_call", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__kvra_call() {
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (g_cuda_stream == nullptr) return nullptr;
  return PyModule_Create(&g_module);
}
