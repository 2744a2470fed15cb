// ck_decode_step for the Python binding without ctypes in between.  The call is made once per
// layer and generated token, and at small batches its marshalling (fifteen tensors, two method
// calls and two ctypes conversions each) took longer than the kernel: 9.9 us from call to call
// for 2 head-problems, B = 256, where the kernel needs 7.1.  The host now needs 5.9 us.
//
// decode_step(entry, shape, 15 tensors, 9 numbers) takes what ck_decode_step takes, `entry` being
// its address.  It returns the status code, or None if any argument is not of the plain
// kind (a contiguous tensor, a number): nothing has been called then, and the caller goes the
// general way, which accepts or refuses the arguments in its own words.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "clusterkv.h"

namespace {

using Entry = decltype(&ck_decode_step);

PyObject *s_is_contiguous, *s_data_ptr;
PyObject* s_shape[7];

bool as_int(PyObject* o, int64_t* v) {
  if (!o || !PyLong_Check(o)) return false;
  int overflow = 0;
  *v = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}
bool as_i32(PyObject* o, int32_t* v) {
  int64_t w;
  if (!as_int(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
  *v = (int32_t)w;
  return true;
}

bool as_pointer(PyObject* t, void** p) {
  if (t == Py_None || PyLong_Check(t)) return false;
  PyObject* c = PyObject_CallMethodNoArgs(t, s_is_contiguous);
  const bool plain = c == Py_True;
  Py_XDECREF(c);
  if (!plain) return false;
  PyObject* a = PyObject_CallMethodNoArgs(t, s_data_ptr);
  int64_t v = 0;
  const bool ok = as_int(a, &v);
  Py_XDECREF(a);
  *p = reinterpret_cast<void*>(static_cast<uintptr_t>(v));
  return ok;
}

bool as_shape(PyObject* o, ck_shape* sh) {
  int32_t* f[7] = {&sh->S, &sh->Hq, &sh->Hkv, &sh->d, nullptr, &sh->C_cap, &sh->dtype};
  for (int i = 0; i < 7; ++i) {
    PyObject* a = PyObject_GetAttr(o, s_shape[i]);
    const bool ok = a && (f[i] ? as_i32(a, f[i]) : as_int(a, &sh->N_cap));
    Py_XDECREF(a);
    if (!ok) return false;
  }
  return true;
}

enum { TENSORS = 15, NUMBERS = 9, ARGS = 2 + TENSORS + NUMBERS };

PyObject* decode_step(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != ARGS) {
    PyErr_SetString(PyExc_TypeError, "decode_step: wrong number of arguments");
    return nullptr;
  }
  int64_t entry;
  ck_shape sh;
  void* p[TENSORS];
  int64_t sink, rb, re, ws_bytes, stream;
  int32_t n_clusters, budget, flags, stride;
  bool ok = as_int(args[0], &entry) && entry != 0 && as_shape(args[1], &sh);
  for (int i = 0; ok && i < TENSORS; ++i) ok = as_pointer(args[2 + i], &p[i]);
  PyObject* const* a = args + 2 + TENSORS;
  ok = ok && as_i32(a[0], &n_clusters) && as_i32(a[1], &budget) && as_i32(a[2], &flags) &&
       as_int(a[3], &sink) && as_int(a[4], &rb) && as_int(a[5], &re) && PyFloat_Check(a[6]) &&
       as_i32(a[7], &stride) && as_int(a[8], &stream);
  if (ok) {
    PyObject* b = PyObject_CallMethod(args[2 + TENSORS - 1], "numel", nullptr);
    ok = as_int(b, &ws_bytes) && ws_bytes >= 0;         // the workspace holds bytes
    Py_XDECREF(b);
  }
  if (!ok) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  const float scale = (float)PyFloat_AS_DOUBLE(a[6]);
  const Entry fn = reinterpret_cast<Entry>(static_cast<uintptr_t>(entry));
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(&sh, p[0], p[1], p[2], p[3], (const int32_t*)p[4], (const int32_t*)p[5],
          (const int32_t*)p[6], n_clusters, budget, (uint32_t)flags, sink, rb, re, scale,
          (float*)p[7], (int32_t*)p[8], (int32_t*)p[9], (int32_t*)p[10], (int32_t*)p[11], stride,
          (int32_t*)p[12], p[13], p[14], (size_t)ws_bytes,
          reinterpret_cast<void*>(static_cast<uintptr_t>(stream)));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(decode_step)),
     METH_FASTCALL, "ck_decode_step on plain tensors; None if an argument is of another kind"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ckhost", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ckhost(void) {
  static const char* const names[7] = {"S", "Hq", "Hkv", "d", "N_cap", "C_cap", "dtype"};
  for (int i = 0; i < 7; ++i)
    if (!(s_shape[i] = PyUnicode_InternFromString(names[i]))) return nullptr;
  if (!(s_is_contiguous = PyUnicode_InternFromString("is_contiguous"))) return nullptr;
  if (!(s_data_ptr = PyUnicode_InternFromString("data_ptr"))) return nullptr;
  return PyModule_Create(&module);
}
