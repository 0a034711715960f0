/* Calls into libsagnn.so from Python: a bound function takes integers (for a pointer Python's own, None, or an object with a
 * buffer, a host array), and returns the C function's int.  Every exported call of the step has only integers and pointers, which go in the same registers and stack
 * slots whatever their width (System V x86-64), so that one call by address serves all of them.  ctypes converts an argument
 * at a time through its type objects: a call of 17 arguments 1.7 us, this way 0.3, of 7.5 for a whole launch. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <stdlib.h>

#if !defined(__x86_64__) || !defined(__linux__)
#error "arguments are passed as the System V x86-64 convention has it"
#endif

#define MOST 24
#define MOST_VIEWS 2
typedef int64_t I;
typedef int (*Fn)(I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I, I);
typedef struct {
  Fn fn;
  PyObject* error;   /* raised for an argument that is none */
  Py_ssize_t n;
  char kind[MOST];   /* 'p' a pointer, 'i' an integer */
} Bound;

static PyObject* call(PyObject* self, PyObject* const* args, Py_ssize_t n) {
  const Bound* b = (const Bound*)PyCapsule_GetPointer(self, NULL);
  if (!b) return NULL;
  if (n != b->n) return PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", n, b->n);
  I v[MOST] = {0};
  Py_buffer views[MOST_VIEWS];
  int n_views = 0, rc;
  PyObject* result = NULL;
  for (Py_ssize_t i = 0; i < n; ++i) {
    if (PyLong_Check(args[i])) {
      v[i] = (I)PyLong_AsUnsignedLongLongMask(args[i]);
    } else if (b->kind[i] == 'i' && PyIndex_Check(args[i])) {
      PyObject* number = PyNumber_Index(args[i]);   /* (an integer of numpy or torch; an array of several has none) */
      if (!number) goto refuse;
      v[i] = (I)PyLong_AsUnsignedLongLongMask(number);
      Py_DECREF(number);
    } else if (b->kind[i] == 'p' && args[i] == Py_None) {
      continue;
    } else if (b->kind[i] == 'p' && n_views < MOST_VIEWS && PyObject_CheckBuffer(args[i])) {
      if (PyObject_GetBuffer(args[i], &views[n_views], PyBUF_ND)) goto refuse;
      if (views[n_views++].ndim == 0) goto refuse;   /* (a number of numpy is no array) */
      v[i] = (I)(uintptr_t)views[n_views - 1].buf;
    } else {
      goto refuse;
    }
    continue;
  refuse:
    PyErr_Clear();
    PyErr_Format(b->error, "argument %zd: an integer expected, or None or an array for a pointer", i + 1);
    goto end;
  }
  Py_BEGIN_ALLOW_THREADS
  rc = b->fn(v[0], v[1], v[2], v[3], v[4], v[5], v[6], v[7], v[8], v[9], v[10], v[11], v[12], v[13], v[14], v[15], v[16], v[17],
             v[18], v[19], v[20], v[21], v[22], v[23]);
  Py_END_ALLOW_THREADS
  result = PyLong_FromLong(rc);
end:
  while (n_views) PyBuffer_Release(&views[--n_views]);
  return result;
}

static PyMethodDef call_def = {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "the bound C function"};

static void drop(PyObject* capsule) {
  Bound* b = (Bound*)PyCapsule_GetPointer(capsule, NULL);
  Py_DECREF(b->error);
  free(b);
}

static PyObject* bind(PyObject* self, PyObject* args) {
  unsigned long long address;
  const char* kinds;
  PyObject* error;
  Py_ssize_t n;
  (void)self;
  if (!PyArg_ParseTuple(args, "Ks#O", &address, &kinds, &n, &error)) return NULL;
  if (!address || n > MOST) return PyErr_Format(PyExc_ValueError, "no address, or more than %d parameters", MOST);
  Bound* b = (Bound*)malloc(sizeof(Bound));
  if (!b) return PyErr_NoMemory();
  b->fn = (Fn)(uintptr_t)address;
  b->error = error;
  Py_INCREF(error);
  b->n = n;
  for (Py_ssize_t i = 0; i < n; ++i) b->kind[i] = kinds[i];
  PyObject* capsule = PyCapsule_New(b, NULL, drop);
  if (!capsule) {
    Py_DECREF(error);
    free(b);
    return NULL;
  }
  PyObject* f = PyCFunction_New(&call_def, capsule);
  Py_DECREF(capsule);
  return f;
}

static PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, "bind(address, kinds, error) -> callable; kinds: a letter per parameter, p pointer, i integer; error: raised for another argument"}, {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", NULL, -1, methods, NULL, NULL, NULL, NULL};
PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
