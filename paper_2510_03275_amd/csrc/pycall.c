/* Calls of the per-token entry points from Python without ctypes' argument
 * conversion (about 2 us a call, as long as one of its two kernel launches).
 * Every argument is a Python integer (pointers as addresses); the functions are
 * taken by address from the library that ctypes has loaded, so this module
 * links against nothing.  The GIL is released around the call, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "../../include/sdq.h"

typedef sdq_status (*linear_fn)(const void*, sdq_dtype, int64_t, const void*, const float*, const sdq_layout*, float*,
                                int32_t, void*, size_t, void*);
typedef sdq_status (*group_fn)(const void*, sdq_dtype, int64_t, int32_t, const void* const*, const float* const*,
                               const sdq_layout*, float* const*, int32_t, void*, size_t, void*);
typedef size_t (*ws_fn)(const sdq_layout*, int64_t);

static linear_fn p_linear;
static group_fn p_group;
static ws_fn p_ws;

/* args[i] as a 64-bit integer; None is 0 (a NULL pointer, the default stream). */
static int take(PyObject* const* args, Py_ssize_t n, Py_ssize_t want, unsigned long long* out) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return -1;
  }
  for (Py_ssize_t i = 0; i < n; ++i) {
    if (args[i] == Py_None) {
      out[i] = 0;
      continue;
    }
    if (!PyLong_Check(args[i])) {
      PyErr_Format(PyExc_TypeError, "argument %zd is not an integer", i);
      return -1;
    }
    out[i] = PyLong_AsUnsignedLongLongMask(args[i]);
  }
  return PyErr_Occurred() ? -1 : 0;
}

static PyObject* py_bind(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  unsigned long long a[3];
  (void)self;
  if (take(args, n, 3, a)) return NULL;
  p_linear = (linear_fn)(uintptr_t)a[0];
  p_group = (group_fn)(uintptr_t)a[1];
  p_ws = (ws_fn)(uintptr_t)a[2];
  Py_RETURN_NONE;
}

#define PTR(T, i) ((T)(uintptr_t)a[i])

static PyObject* py_linear(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  unsigned long long a[11];
  sdq_status st;
  (void)self;
  if (take(args, n, 11, a)) return NULL;
  Py_BEGIN_ALLOW_THREADS
  st = p_linear(PTR(const void*, 0), (sdq_dtype)a[1], (int64_t)a[2], PTR(const void*, 3), PTR(const float*, 4),
                PTR(const sdq_layout*, 5), PTR(float*, 6), (int32_t)a[7], PTR(void*, 8), (size_t)a[9],
                PTR(void*, 10));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

static PyObject* py_group(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  unsigned long long a[12];
  sdq_status st;
  (void)self;
  if (take(args, n, 12, a)) return NULL;
  Py_BEGIN_ALLOW_THREADS
  st = p_group(PTR(const void*, 0), (sdq_dtype)a[1], (int64_t)a[2], (int32_t)a[3], PTR(const void* const*, 4),
               PTR(const float* const*, 5), PTR(const sdq_layout*, 6), PTR(float* const*, 7), (int32_t)a[8],
               PTR(void*, 9), (size_t)a[10], PTR(void*, 11));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

static PyObject* py_ws(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  unsigned long long a[2];
  (void)self;
  if (take(args, n, 2, a)) return NULL;
  return PyLong_FromSize_t(p_ws(PTR(const sdq_layout*, 0), (int64_t)a[1]));
}

static PyMethodDef methods[] = {
    {"bind", (PyCFunction)(void (*)(void))py_bind, METH_FASTCALL, "addresses of the library's functions"},
    {"linear", (PyCFunction)(void (*)(void))py_linear, METH_FASTCALL, "sdq_linear"},
    {"linear_group", (PyCFunction)(void (*)(void))py_group, METH_FASTCALL, "sdq_linear_group"},
    {"linear_workspace_bytes", (PyCFunction)(void (*)(void))py_ws, METH_FASTCALL, "sdq_linear_workspace_bytes"},
    {NULL, NULL, 0, NULL},
};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_sdqcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__sdqcall(void) { return PyModule_Create(&module); }
