/* The per-token call of the Python binding without ctypes, whose conversion of nine arguments costs the host more than the
 * checks and the choice of a kernel behind them (a call that fails the first check: 0.42 us, 0.06 so, on one host, 1.25 and 0.12 on
 * another).  A decode call of a small layer is bound by the host: 128 x 205 fp32 4.8 -> 4.1 us, a prompt and 16 tokens of 256 x 1024
 * 137 -> 126. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "coreinfer.h"

static int pointer(PyObject* o, void** out) {
  *out = o == Py_None ? NULL : PyLong_AsVoidPtr(o);
  return *out != NULL || !PyErr_Occurred();
}

static int number(PyObject* o, long long* out) {
  *out = PyLong_AsLongLong(o);
  return *out != -1 || !PyErr_Occurred();
}

/* ffn_decode(x, B, weights, dtype, act, y, ws, ws_bytes, stream) -> status; addresses are integers or None */
static PyObject* ffn_decode(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void *x, *w, *y, *ws, *stream;
  long long B, dtype, act, bytes;
  int status;
  (void)self;
  if (n != 9) {
    PyErr_SetString(PyExc_TypeError, "nine arguments");
    return NULL;
  }
  if (!pointer(a[0], &x) || !number(a[1], &B) || !pointer(a[2], &w) || !number(a[3], &dtype) || !number(a[4], &act) ||
      !pointer(a[5], &y) || !pointer(a[6], &ws) || !number(a[7], &bytes) || !pointer(a[8], &stream))
    return NULL;
  Py_BEGIN_ALLOW_THREADS
  status = coreinfer_ffn_decode(x, B, (const ci_ffn_weights*)w, (int)dtype, (int)act, y, ws, (size_t)bytes, stream);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {{"ffn_decode", (PyCFunction)(void (*)(void))ffn_decode, METH_FASTCALL, NULL}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
