// Argument marshalling of the device entry points for CPython: what the ctypes functions of lutgemm.py do, for the
// arguments a program usually has (tensors, integers).  A call of a small layer is bound by the host: back to back,
// with the stream looked up each time (2.7 us), 1024 x 1024 took 7.5 us from Python before this and takes 6.4 (4.9 on the
// device; of the host's time 2.2 are the launch itself).  Anything else (keywords, numbers that are not plain ints, other buffer objects, wrong counts, a
// library that is not loaded yet) goes to the ctypes function of the same name, which has the last word on what is
// accepted and what is raised.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <climits>
#include <cstddef>
#include <cstdint>

namespace {

typedef int (*GemvFn)(const void*, const void*, const void*, const void*, void*, int, int, int, int64_t, int64_t, unsigned, void*, size_t,
                      void*);
typedef int (*GemmFn)(const void*, const void*, const void*, const void*, void*, int, int, int, int64_t, int64_t, int, unsigned, void*,
                      size_t, void*);
typedef int (*StaticFn)(const void*, const void*, const void*, const void*, void*, int, int, int, int64_t, int64_t, unsigned, void*);
typedef int (*GroupFn)(const void* const*, const void* const*, const void* const*, const void* const*, void* const*, const int64_t*,
                       const int64_t*, int, int, int, int, unsigned, void*, size_t, void*);

enum Which { kGemv, kGemm, kMfma, kDequant, kStatic, kGroup, kCount };
const char* const kNames[kCount] = {"lutgemm_gemv", "lutgemm_gemm", "lutgemm_gemm_mfma", "lutgemm_gemm_dequant_mfma", "lutgemm_gemv_static",
                                    "lutgemm_gemv_group"};

void* g_function[kCount];        // of the loaded library, null until then
PyObject* g_ctypes[kCount];      // lutgemm.py's functions
PyObject* g_check;               // lutgemm.py's _check(code, where): raises
PyObject* g_data_ptr;            // "data_ptr"

// The converters return false, with no exception set, where ctypes is to decide.
bool address(PyObject* o, void** out) {
  if (o == Py_None) {
    *out = nullptr;
    return true;
  }
  PyObject* number = o;
  if (!PyLong_CheckExact(o)) {
    number = PyObject_VectorcallMethod(g_data_ptr, &o, 1 | PY_VECTORCALL_ARGUMENTS_OFFSET, nullptr);
    if (!number) {
      PyErr_Clear();
      return false;
    }
  }
  bool ok = PyLong_CheckExact(number);
  if (ok) {
    const unsigned long long v = PyLong_AsUnsignedLongLong(number);
    if (v == (unsigned long long)-1 && PyErr_Occurred()) {
      PyErr_Clear();
      ok = false;
    }
    *out = reinterpret_cast<void*>((uintptr_t)v);
  }
  if (number != o) Py_DECREF(number);
  return ok;
}

bool integer(PyObject* o, int64_t lowest, int64_t highest, int64_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow != 0 || v < lowest || v > highest) return false;
  *out = v;
  return true;
}
bool c_int(PyObject* o, int* out) {
  int64_t v;
  if (!integer(o, INT_MIN, INT_MAX, &v)) return false;
  *out = (int)v;
  return true;
}

PyObject* by_ctypes(Which w, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  if (!g_ctypes[w]) {
    PyErr_SetString(PyExc_RuntimeError, "the binding has not been set up");
    return nullptr;
  }
  return PyObject_Vectorcall(g_ctypes[w], args, (size_t)nargs, kwnames);
}

PyObject* result(Which w, int code) {
  if (code == 0) Py_RETURN_NONE;
  return PyObject_CallFunction(g_check, "is", code, kNames[w]);
}

// x, bits, alpha, z, y, q, g, mu, m, n, [batch,] flags, [workspace, workspace_bytes,] stream=0
PyObject* one_layer(Which w, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  const bool batched = w == kGemm || w == kMfma || w == kDequant, scratch = w != kStatic;
  const Py_ssize_t needed = 11 + (batched ? 1 : 0) + (scratch ? 2 : 0);
  if (!g_function[w] || (kwnames && PyTuple_GET_SIZE(kwnames) != 0) || (nargs != needed && nargs != needed + 1))
    return by_ctypes(w, args, nargs, kwnames);
  void *buf[5], *ws = nullptr, *stream = nullptr;
  int q, g, mu, batch = 1;
  int64_t m, n, flags, bytes = 0;
  bool ok = true;
  for (int i = 0; i < 5 && ok; ++i) ok = address(args[i], &buf[i]);
  ok = ok && c_int(args[5], &q) && c_int(args[6], &g) && c_int(args[7], &mu) && integer(args[8], INT64_MIN, INT64_MAX, &m) &&
       integer(args[9], INT64_MIN, INT64_MAX, &n);
  Py_ssize_t at = 10;
  if (batched) ok = ok && c_int(args[at++], &batch);
  ok = ok && integer(args[at++], 0, UINT_MAX, &flags);
  if (scratch) {
    ok = ok && address(args[at], &ws) && integer(args[at + 1], 0, INT64_MAX, &bytes);
    at += 2;
  }
  if (nargs > needed) ok = ok && PyLong_CheckExact(args[at]) && address(args[at], &stream);
  if (!ok) return by_ctypes(w, args, nargs, kwnames);
  int code;
  Py_BEGIN_ALLOW_THREADS
  if (batched)
    code = reinterpret_cast<GemmFn>(g_function[w])(buf[0], buf[1], buf[2], buf[3], buf[4], q, g, mu, m, n, batch, (unsigned)flags, ws,
                                                   (size_t)bytes, stream);
  else if (scratch)
    code = reinterpret_cast<GemvFn>(g_function[w])(buf[0], buf[1], buf[2], buf[3], buf[4], q, g, mu, m, n, (unsigned)flags, ws,
                                                   (size_t)bytes, stream);
  else
    code = reinterpret_cast<StaticFn>(g_function[w])(buf[0], buf[1], buf[2], buf[3], buf[4], q, g, mu, m, n, (unsigned)flags, stream);
  Py_END_ALLOW_THREADS
  return result(w, code);
}

constexpr Py_ssize_t kMostLayers = 8;

bool list_of(PyObject* o, Py_ssize_t count, PyObject** items) {
  if (!(PyList_CheckExact(o) || PyTuple_CheckExact(o)) || PySequence_Fast_GET_SIZE(o) != count) return false;
  for (Py_ssize_t i = 0; i < count; ++i) items[i] = PySequence_Fast_GET_ITEM(o, i);
  return true;
}

// x, bits, alpha, z, y, m, n, q, g, mu, flags, workspace, workspace_bytes, stream=0
PyObject* group(PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  const Which w = kGroup;
  if (!g_function[w] || (kwnames && PyTuple_GET_SIZE(kwnames) != 0) || (nargs != 13 && nargs != 14) ||
      !(PyList_CheckExact(args[5]) || PyTuple_CheckExact(args[5])))
    return by_ctypes(w, args, nargs, kwnames);
  const Py_ssize_t count = PySequence_Fast_GET_SIZE(args[5]);
  void *buf[5][kMostLayers], *ws, *stream = nullptr;
  int64_t shape[2][kMostLayers], flags, bytes;
  int q, g, mu;
  PyObject* items[kMostLayers];
  bool ok = count <= kMostLayers;
  // Every item is held while the lists' owners may run (data_ptr of an object of Python's could change a list).
  for (int b = 0; b < 5 && ok; ++b) {
    if (b == 3 && args[b] == Py_None) continue;
    ok = list_of(args[b], count, items);
    if (!ok) break;
    for (Py_ssize_t i = 0; i < count; ++i) Py_INCREF(items[i]);
    for (Py_ssize_t i = 0; i < count && ok; ++i) ok = address(items[i], &buf[b][i]);
    for (Py_ssize_t i = 0; i < count; ++i) Py_DECREF(items[i]);
  }
  for (int b = 0; b < 2 && ok; ++b) {
    ok = list_of(args[5 + b], count, items);
    for (Py_ssize_t i = 0; i < count && ok; ++i) ok = integer(items[i], INT64_MIN, INT64_MAX, &shape[b][i]);
  }
  ok = ok && c_int(args[7], &q) && c_int(args[8], &g) && c_int(args[9], &mu) && integer(args[10], 0, UINT_MAX, &flags) &&
       address(args[11], &ws) && integer(args[12], 0, INT64_MAX, &bytes);
  if (nargs == 14) ok = ok && PyLong_CheckExact(args[13]) && address(args[13], &stream);
  if (!ok) return by_ctypes(w, args, nargs, kwnames);
  int code;
  Py_BEGIN_ALLOW_THREADS
  code = reinterpret_cast<GroupFn>(g_function[w])(buf[0], buf[1], buf[2], args[3] == Py_None ? nullptr : buf[3], buf[4], shape[0], shape[1],
                                                  (int)count, q, g, mu, (unsigned)flags, ws, (size_t)bytes, stream);
  Py_END_ALLOW_THREADS
  return result(w, code);
}

template <Which W>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  return W == kGroup ? group(args, nargs, kwnames) : one_layer(W, args, nargs, kwnames);
}

// set_up(functions by name, check): the ctypes functions and what raises; load(addresses by name): the library's functions.
PyObject* set_up(PyObject*, PyObject* args) {
  PyObject *functions, *check;
  if (!PyArg_ParseTuple(args, "O!O", &PyDict_Type, &functions, &check)) return nullptr;
  for (int w = 0; w < kCount; ++w) {
    PyObject* f = PyDict_GetItemString(functions, kNames[w]);
    if (!f) {
      PyErr_SetString(PyExc_KeyError, kNames[w]);
      return nullptr;
    }
    Py_INCREF(f);
    Py_XSETREF(g_ctypes[w], f);
  }
  Py_INCREF(check);
  Py_XSETREF(g_check, check);
  Py_RETURN_NONE;
}

PyObject* load(PyObject*, PyObject* args) {
  PyObject* addresses;
  if (!PyArg_ParseTuple(args, "O!", &PyDict_Type, &addresses)) return nullptr;
  for (int w = 0; w < kCount; ++w) {
    PyObject* a = PyDict_GetItemString(addresses, kNames[w]);   // (a host-only build of the library has none: ctypes then says so)
    void* p = nullptr;
    if (a && !address(a, &p)) {
      PyErr_SetString(PyExc_TypeError, "an address is a non-negative int");
      return nullptr;
    }
    g_function[w] = p;
  }
  Py_RETURN_NONE;
}

#define LAYER_ARGS "x, bits, alpha, z, y, q, g, mu, m, n, "
#define ENTRY(name, which, signature) \
  {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(entry<which>)), METH_FASTCALL | METH_KEYWORDS, name "(" signature ")\n--\n\n"}
PyMethodDef g_methods[] = {
    ENTRY("lutgemm_gemv", kGemv, LAYER_ARGS "flags, workspace, workspace_bytes, stream=0"),
    ENTRY("lutgemm_gemm", kGemm, LAYER_ARGS "batch, flags, workspace, workspace_bytes, stream=0"),
    ENTRY("lutgemm_gemm_mfma", kMfma, LAYER_ARGS "batch, flags, workspace, workspace_bytes, stream=0"),
    ENTRY("lutgemm_gemm_dequant_mfma", kDequant, LAYER_ARGS "batch, flags, workspace, workspace_bytes, stream=0"),
    ENTRY("lutgemm_gemv_static", kStatic, LAYER_ARGS "flags, stream=0"),
    ENTRY("lutgemm_gemv_group", kGroup, "x, bits, alpha, z, y, m, n, q, g, mu, flags, workspace, workspace_bytes, stream=0"),
    {"set_up", set_up, METH_VARARGS, nullptr},
    {"load", load, METH_VARARGS, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  g_data_ptr = PyUnicode_InternFromString("data_ptr");
  return g_data_ptr ? PyModule_Create(&g_module) : nullptr;
}
