// The calls of a step from Python: tensors and lists of them into raw addresses and pointer arrays, then the call, without the GIL.
//
// ctypes builds an array object for every list and converts every argument by its type: a step's four calls took 17.4 us of host time where the
// library itself takes 10, more than the kernels of a small state run.  Here they take 10.2 with the one launch less of an update that derives its
// constants: a step of 0.8 M parameters 16.1 -> 13.9 us, of 0.1 M 14.5 -> 9.9.  What a call is handed in another form than the
// usual one (an argument type not named below) is left to ctypes: the function returns None and has done nothing.  The lists come last, since
// their addresses are what a call takes time for: 100 tensors by ctypes 45 us, here 16; both, one behind the other, 58.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>
#include <cstring>
#include <limits>
#include <new>
#include <vector>

#include "ptchunk.h"

namespace {

// Entry points of the loaded libptchunk.so, in the order bind() takes them.
struct Entry {
  int (*pack)(pt_ctx*, const pt_pack_plan*, void* const*, void*);
  int (*unpack)(pt_ctx*, const pt_pack_plan*, const void* const*, void*);
  int (*accum)(pt_ctx*, const pt_pack_plan*, float* const*, int, int, void*);
  int (*sqnorm)(pt_ctx*, const void* const*, uint32_t, uint32_t, int, void*);
  int (*update)(pt_ctx*, const pt_hparams*, uint32_t, uint32_t, const void* const*, float* const*, float* const*, float* const*,
                void* const*, void*);
  int (*step_end)(pt_ctx*, void*);
  int (*noalloc)(const void*, int, uint64_t, uint32_t, double, double*, int32_t*, void*);
} entry = {};
constexpr size_t N_ENTRIES = sizeof(Entry) / sizeof(void*);
PyTypeObject *handle_type = nullptr, *hparams_type = nullptr;      // ctypes.c_void_p, binding.pt_hparams
PyObject *initialized = nullptr, *get_device = nullptr, *raw_stream = nullptr;     // torch's, for the current stream; raw_stream may be None
PyObject *s_data_ptr = nullptr, *s_value = nullptr, *s_cuda_stream = nullptr;

// Each returns false, with no Python error set or with the one a callee has raised, where it does not know the form.
bool as_address(PyObject* x, void** out) {
  if (PyLong_CheckExact(x)) {
    *out = PyLong_AsVoidPtr(x);
    if (!PyErr_Occurred()) return true;
    PyErr_Clear();
  }
  return false;
}

bool as_handle(PyObject* x, void** out) {
  if (Py_TYPE(x) != handle_type) return false;
  PyObject* v = PyObject_GetAttr(x, s_value);
  if (!v) return false;
  const bool ok = v != Py_None && as_address(v, out);      // a NULL handle is ctypes' to pass on
  Py_DECREF(v);
  return ok;
}

bool tensor_address(PyObject* x, void** out) {
  PyObject* v = PyObject_CallMethodNoArgs(x, s_data_ptr);
  if (!v) return false;
  const bool ok = as_address(v, out);
  Py_DECREF(v);
  return ok;
}

// A list of tensors, addresses and None into `out`, which holds one NULL for an empty one.
bool is_array(PyObject* list) { return PyList_CheckExact(list); }
bool as_array(PyObject* list, std::vector<void*>& out) try {
  if (!is_array(list)) return false;
  out.reserve(size_t(PyList_GET_SIZE(list)) + 1);
  for (Py_ssize_t i = 0; i < PyList_GET_SIZE(list); ++i) {
    PyObject* x = PyList_GET_ITEM(list, i);
    void* p = nullptr;
    if (x != Py_None) {
      Py_INCREF(x);
      const bool ok = PyLong_Check(x) ? as_address(x, &p) : tensor_address(x, &p);
      Py_DECREF(x);
      if (!ok) return false;
    }
    out.push_back(p);
  }
  if (out.empty()) out.push_back(nullptr);
  return true;
} catch (const std::bad_alloc&) {
  PyErr_NoMemory();
  return false;
}

template <class T>
bool as_number(PyObject* x, T* out) {
  if (!PyLong_Check(x)) return false;                      // True and False too
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(x, &overflow);
  if (overflow || v < 0 || uint64_t(v) > uint64_t(std::numeric_limits<T>::max())) return false;
  *out = T(v);
  return true;
}

// None: torch's current stream; a stream object: its handle.
bool as_stream(PyObject* x, void** out) {
  if (PyLong_Check(x)) return as_address(x, out);
  if (x != Py_None) {
    PyObject* v = PyObject_GetAttr(x, s_cuda_stream);
    if (!v) {
      if (PyErr_ExceptionMatches(PyExc_AttributeError)) PyErr_Clear();      // no stream: ctypes' route says so
      return false;
    }
    const bool ok = as_address(v, out);
    Py_DECREF(v);
    return ok;
  }
  if (raw_stream == Py_None) return false;
  PyObject* is = PyObject_CallNoArgs(initialized);
  if (!is) return false;
  const bool yes = is == Py_True;
  Py_DECREF(is);
  if (!yes) return false;
  PyObject* dev = PyObject_CallNoArgs(get_device);
  PyObject* s = dev ? PyObject_CallOneArg(raw_stream, dev) : nullptr;
  Py_XDECREF(dev);
  if (!s) return false;
  const bool ok = as_address(s, out);
  Py_DECREF(s);
  return ok;
}

PyObject* not_here() {
  if (PyErr_Occurred()) return nullptr;
  Py_RETURN_NONE;
}

template <class F>
PyObject* run(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

PyObject* pack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *plan, *st;
  std::vector<void*> p;
  if (n != 4 || !as_handle(a[0], &ctx) || !as_handle(a[1], &plan) || !as_stream(a[3], &st) || !as_array(a[2], p)) return not_here();
  return run([&] { return entry.pack((pt_ctx*)ctx, (const pt_pack_plan*)plan, p.data(), st); });
}

PyObject* unpack(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *plan, *st;
  std::vector<void*> p;
  if (n != 4 || !as_handle(a[0], &ctx) || !as_handle(a[1], &plan) || !as_stream(a[3], &st) || !as_array(a[2], p)) return not_here();
  return run([&] { return entry.unpack((pt_ctx*)ctx, (const pt_pack_plan*)plan, p.data(), st); });
}

PyObject* accum(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *plan, *st;
  std::vector<void*> p;
  int over, norm;
  if (n != 6 || !as_handle(a[0], &ctx) || !as_handle(a[1], &plan) || !as_number(a[3], &over) || !as_number(a[4], &norm) ||
      !as_stream(a[5], &st) || !as_array(a[2], p))
    return not_here();
  return run([&] { return entry.accum((pt_ctx*)ctx, (const pt_pack_plan*)plan, (float* const*)p.data(), over != 0, norm != 0, st); });
}

PyObject* sqnorm(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *st;
  std::vector<void*> p;
  uint32_t first, count;
  int how;
  if (n != 6 || !as_handle(a[0], &ctx) || !as_number(a[2], &first) || !as_number(a[3], &count) || !as_number(a[4], &how) ||
      !as_stream(a[5], &st) || (a[1] != Py_None && !as_array(a[1], p)))
    return not_here();
  return run([&] { return entry.sqnorm((pt_ctx*)ctx, p.empty() ? nullptr : p.data(), first, count, how, st); });
}

PyObject* update(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *st;
  std::vector<void*> p[5];
  uint32_t first, count;
  if (n != 10 || !as_handle(a[0], &ctx) || Py_TYPE(a[1]) != hparams_type || !as_number(a[2], &first) || !as_number(a[3], &count))
    return not_here();
  for (int k = 0; k < 5; ++k)
    if (!is_array(a[4 + k])) return not_here();
  pt_hparams hp;
  Py_buffer b;
  if (!as_stream(a[9], &st) || PyObject_GetBuffer(a[1], &b, PyBUF_SIMPLE) != 0) return not_here();
  std::memcpy(&hp, b.buf, sizeof hp);                      // hparams_type has its size (bind)
  PyBuffer_Release(&b);
  for (int k = 0; k < 5; ++k)
    if (!as_array(a[4 + k], p[k])) return not_here();
  return run([&] {
    return entry.update((pt_ctx*)ctx, &hp, first, count, p[0].data(), (float* const*)p[1].data(), (float* const*)p[2].data(),
                        (float* const*)p[3].data(), p[4].data(), st);
  });
}

PyObject* step_end(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *ctx, *st;
  if (n != 2 || !as_handle(a[0], &ctx) || !as_stream(a[1], &st)) return not_here();
  return run([&] { return entry.step_end((pt_ctx*)ctx, st); });
}

PyObject* noalloc(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void *g, *out, *inf, *st;
  int dtype;
  uint64_t elems;
  uint32_t chunks;
  if (n != 8 || !as_number(a[1], &dtype) || !as_number(a[2], &elems) || !as_number(a[3], &chunks) || !PyFloat_CheckExact(a[4])) return not_here();
  const double scale = PyFloat_AS_DOUBLE(a[4]);
  if (PyLong_Check(a[0]) || PyLong_Check(a[5]) || PyLong_Check(a[6]) || a[0] == Py_None || a[5] == Py_None || a[6] == Py_None) return not_here();
  if (!as_stream(a[7], &st) || !tensor_address(a[0], &g) || !tensor_address(a[5], &out) || !tensor_address(a[6], &inf)) return not_here();
  return run([&] { return entry.noalloc(g, dtype, elems, chunks, scale, (double*)out, (int32_t*)inf, st); });
}

// bind(addresses of the entry points, c_void_p, pt_hparams, is_initialized, getDevice, getCurrentRawStream or None)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *list, *ht, *hp, *is, *dev, *raw;
  if (!PyArg_ParseTuple(args, "O!O!O!OOO", &PyList_Type, &list, &PyType_Type, &ht, &PyType_Type, &hp, &is, &dev, &raw)) return nullptr;
  if (PyList_GET_SIZE(list) != Py_ssize_t(N_ENTRIES)) return PyErr_Format(PyExc_ValueError, "bind: %zu entry points", N_ENTRIES);
  void* at[N_ENTRIES];
  for (size_t i = 0; i < N_ENTRIES; ++i)
    if (!(at[i] = PyLong_AsVoidPtr(PyList_GET_ITEM(list, Py_ssize_t(i))))) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "bind: NULL");
  PyObject* one = PyObject_CallNoArgs(hp);
  Py_buffer b;
  if (!one || PyObject_GetBuffer(one, &b, PyBUF_SIMPLE) != 0) { Py_XDECREF(one); return nullptr; }
  const Py_ssize_t size = b.len;
  PyBuffer_Release(&b);
  Py_DECREF(one);
  if (size != Py_ssize_t(sizeof(pt_hparams))) return PyErr_Format(PyExc_ValueError, "bind: pt_hparams of %zd bytes, built with %zu", size, sizeof(pt_hparams));
  std::memcpy(&entry, at, sizeof entry);
  for (PyObject* o : {ht, hp, is, dev, raw}) Py_INCREF(o);      // kept as long as the process
  handle_type = (PyTypeObject*)ht; hparams_type = (PyTypeObject*)hp;
  initialized = is; get_device = dev; raw_stream = raw;
  Py_RETURN_NONE;
}

#define PT_FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, PT_FAST(pack), PT_FAST(unpack), PT_FAST(accum), PT_FAST(sqnorm),
                         PT_FAST(update), PT_FAST(step_end), PT_FAST(noalloc), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ptcall", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ptcall(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_value = PyUnicode_InternFromString("value");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return s_data_ptr && s_value && s_cuda_stream ? PyModule_Create(&module) : nullptr;
}
