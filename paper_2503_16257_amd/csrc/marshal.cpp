// The per-layer calls of the binding, marshalled natively: a decode step makes one call per layer, and in
// Python the checks and pointers of its tensors cost 2 us and more of it (both sides in binding.py).
//
// What a call does is what binding.py does for it - tensor type, device, contiguity and dtype checked, then the
// C entry point - for plain torch.Tensor arguments that pass and structures of binding.py's own classes; anything
// else returns None, and binding.py's own path takes the call and raises what it always raised.  Nothing is kept
// between calls but the entry points' addresses and the two classes, which bind() hands over once.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include "../../include/vidkv.h"

namespace {

decltype(&vidkv_decode_attention) g_decode;
decltype(&vidkv_decode_attention_noalloc) g_decode_noalloc;
decltype(&vidkv_flush_residual) g_flush;
PyTypeObject* g_params_type;         // binding.VidkvParams
PyTypeObject* g_side_type;           // binding.VidkvSideStream

// Memory of a ctypes structure of class `type` and exactly `size` bytes (ctypes refuses other objects, whatever
// buffer they have).
class Struct {
 public:
  Struct(PyObject* o, PyTypeObject* type, size_t size) {
    if (!PyObject_TypeCheck(o, type)) return;
    if (PyObject_GetBuffer(o, &view_, PyBUF_SIMPLE) != 0) { PyErr_Clear(); return; }
    held_ = true;
    if ((size_t)view_.len == size) ptr_ = view_.buf;
  }
  ~Struct() { if (held_) PyBuffer_Release(&view_); }
  Struct(const Struct&) = delete;
  const void* get() const { return ptr_; }

 private:
  Py_buffer view_;
  bool held_ = false;
  const void* ptr_ = nullptr;
};

// Data pointer (and size) of a contiguous device tensor of type t; None gives NULL where that is allowed.
bool tensor(PyObject* o, c10::ScalarType t, bool none_ok, void** ptr, size_t* bytes = nullptr) {
  *ptr = nullptr;
  if (o == Py_None) return none_ok;
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& x = THPVariable_Unpack(o);
  if (!x.defined() || !x.has_storage() || !x.is_cuda() || x.scalar_type() != t || !x.is_contiguous()) return false;
  *ptr = x.data_ptr();
  if (bytes) *bytes = x.nbytes();
  return true;
}

bool integer(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int over = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &over);
  if (over || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

bool handle(PyObject* o, void** v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsVoidPtr(o);
  if (PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}

// The stream's handle, asked for when the other arguments have passed: fn(stream).  -1: a Python error is set.
int stream_handle(PyObject* fn, PyObject* stream, void** v) {
  PyObject* h = PyObject_CallFunctionObjArgs(fn, stream, nullptr);
  if (!h) return -1;
  const bool ok = handle(h, v);
  Py_DECREF(h);
  return ok;
}

// f() may throw (a tensor without data): then the Python path takes the call
template <class F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// (params, layer, q, packed_K, packed_V, K_tail, V_tail, tail_capacity, tail_len, out, workspace, stream function, stream, side or None)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 14 || !g_decode) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    int32_t layer, cap;
    void *q, *pk, *pv, *kt, *vt, *tl, *out, *ws, *stream;
    size_t wsb = 0;
    if (!integer(a[1], &layer) || !tensor(a[2], at::kHalf, true, &q) || !tensor(a[3], at::kByte, true, &pk) ||
        !tensor(a[4], at::kByte, true, &pv) || !tensor(a[5], at::kHalf, true, &kt) || !tensor(a[6], at::kHalf, true, &vt) ||
        !integer(a[7], &cap) || !tensor(a[8], at::kInt, true, &tl) || !tensor(a[9], at::kHalf, true, &out) ||
        !tensor(a[10], at::kByte, false, &ws, &wsb))
      Py_RETURN_NONE;
    const Struct p(a[0], g_params_type, sizeof(vidkv_params));
    if (!p.get()) Py_RETURN_NONE;
    vidkv_side_stream side;
    const bool has_side = a[13] != Py_None;
    if (has_side) {
      const Struct s(a[13], g_side_type, sizeof(side));
      if (!s.get()) Py_RETURN_NONE;
      side = *static_cast<const vidkv_side_stream*>(s.get());
    }
    const int got = stream_handle(a[11], a[12], &stream);
    if (got < 0) return nullptr;
    if (!got) Py_RETURN_NONE;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = g_decode(static_cast<const vidkv_params*>(p.get()), layer, q, pk, pv, kt, vt, cap, static_cast<const int32_t*>(tl),
                  out, ws, wsb, stream, has_side ? &side : nullptr);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  });
}

// (params, layer, q, packed_K, packed_V, K_tail, V_tail, tail_capacity, tail_len, out, stream function, stream)
PyObject* decode_noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12 || !g_decode_noalloc) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    int32_t layer, cap;
    void *q, *pk, *pv, *kt, *vt, *tl, *out, *stream;
    if (!integer(a[1], &layer) || !tensor(a[2], at::kHalf, true, &q) || !tensor(a[3], at::kByte, true, &pk) ||
        !tensor(a[4], at::kByte, true, &pv) || !tensor(a[5], at::kHalf, true, &kt) || !tensor(a[6], at::kHalf, true, &vt) ||
        !integer(a[7], &cap) || !tensor(a[8], at::kInt, true, &tl) || !tensor(a[9], at::kHalf, true, &out))
      Py_RETURN_NONE;
    const Struct p(a[0], g_params_type, sizeof(vidkv_params));
    if (!p.get()) Py_RETURN_NONE;
    const int got = stream_handle(a[10], a[11], &stream);
    if (got < 0) return nullptr;
    if (!got) Py_RETURN_NONE;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = g_decode_noalloc(static_cast<const vidkv_params*>(p.get()), layer, q, pk, pv, kt, vt, cap,
                          static_cast<const int32_t*>(tl), out, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  });
}

// (params, layer, K_tail, V_tail, tail_capacity, n_flush, packed_K, packed_V, stream function, stream)
PyObject* flush(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10 || !g_flush) Py_RETURN_NONE;
  return guarded([&]() -> PyObject* {
    int32_t layer, cap, nf;
    void *kt, *vt, *pk, *pv, *stream;
    size_t kb = 0, vb = 0;
    if (!integer(a[1], &layer) || !tensor(a[2], at::kHalf, true, &kt) || !tensor(a[3], at::kHalf, true, &vt) ||
        !integer(a[4], &cap) || !integer(a[5], &nf) || !tensor(a[6], at::kByte, false, &pk, &kb) ||
        !tensor(a[7], at::kByte, false, &pv, &vb))
      Py_RETURN_NONE;
    const Struct p(a[0], g_params_type, sizeof(vidkv_params));
    if (!p.get()) Py_RETURN_NONE;
    const int got = stream_handle(a[8], a[9], &stream);
    if (got < 0) return nullptr;
    if (!got) Py_RETURN_NONE;
    int st;
    Py_BEGIN_ALLOW_THREADS
    st = g_flush(static_cast<const vidkv_params*>(p.get()), layer, kt, vt, cap, nf, pk, kb, pv, vb, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(st);
  });
}

// (addresses of vidkv_decode_attention, vidkv_decode_attention_noalloc, vidkv_flush_residual; the classes of
// vidkv_params and vidkv_side_stream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* f[3];
  if (n != 5 || !handle(a[0], &f[0]) || !handle(a[1], &f[1]) || !handle(a[2], &f[2]) || !PyType_Check(a[3]) ||
      !PyType_Check(a[4])) {
    PyErr_SetString(PyExc_TypeError, "bind: three addresses and two classes");
    return nullptr;
  }
  Py_INCREF(a[3]);                                     // (kept, with the module, for as long as the process)
  Py_INCREF(a[4]);
  g_params_type = reinterpret_cast<PyTypeObject*>(a[3]);
  g_side_type = reinterpret_cast<PyTypeObject*>(a[4]);
  g_decode = reinterpret_cast<decltype(g_decode)>(f[0]);
  g_decode_noalloc = reinterpret_cast<decltype(g_decode_noalloc)>(f[1]);
  g_flush = reinterpret_cast<decltype(g_flush)>(f[2]);
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"decode_attention", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(decode)), METH_FASTCALL, nullptr},
    {"decode_attention_noalloc", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(decode_noalloc)), METH_FASTCALL, nullptr},
    {"flush_residual", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(flush)), METH_FASTCALL, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(bind)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "vidkv_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// built_for: the Python and the torch that this was compiled against (binding.py uses it with no other)
PyMODINIT_FUNC PyInit_vidkv_marshal(void) {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "built_for", VIDKV_BUILT_FOR) != 0) Py_CLEAR(m);
  return m;
}
