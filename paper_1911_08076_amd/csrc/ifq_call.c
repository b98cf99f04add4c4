/* CPython entry to the launching functions of libifq.so: the arguments of one
 * call are taken from the interpreter's array and passed on with their C
 * types, the GIL released meanwhile.
 *
 * On a small layer the caller's thread, not the GPU, sets the rate: through
 * ctypes a call spent 3-5 us converting ten arguments (0.5 us each for a
 * tensor's address), as long as the kernel it launches.
 *
 * A tensor argument is None (NULL) or an object with data_ptr() (a torch
 * tensor), an integer an int; anything else goes through the binding's own
 * conversions, which take and refuse what ctypes takes and refuses.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

#include "ifq.h"

static struct {
  __typeof__(&ifq_conv_forward) conv_forward;
  __typeof__(&ifq_conv_forward_fp4) conv_forward_fp4;
  __typeof__(&ifq_conv_pool_forward) conv_pool_forward;
  __typeof__(&ifq_conv_pool_forward_fp4) conv_pool_forward_fp4;
  __typeof__(&ifq_maxpool_codes) maxpool_codes;
  __typeof__(&ifq_convert_codes) convert_codes;
  __typeof__(&ifq_run_stack) run_stack;
  __typeof__(&ifq_run_stack_static) run_stack_static;
} fn;
static PyObject* s_data_ptr;   /* "data_ptr" */
static PyObject* conv_ptr;     /* the binding's conversion of other tensor arguments */
static PyObject* conv_int;     /* and of other integers */

/* The address of a tensor argument; 0 on success. */
static int address(PyObject* o, int64_t* v) {
  if (o == Py_None) {
    *v = 0;
    return 0;
  }
  PyObject* r = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!r && PyErr_ExceptionMatches(PyExc_AttributeError) && conv_ptr) {
    PyErr_Clear();
    r = PyObject_CallOneArg(conv_ptr, o);
  }
  if (!r) return -1;
  *v = (int64_t)PyLong_AsUnsignedLongLongMask(r);
  Py_DECREF(r);
  return PyErr_Occurred() ? -1 : 0;
}

/* The low 64 bits of an integer argument; 0 on success. */
static int integer(PyObject* o, int64_t* v) {
  if (PyLong_Check(o)) {
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(o);
  } else {
    PyObject* r = conv_int ? PyObject_CallOneArg(conv_int, o) : NULL;
    if (!r) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "an int is required");
      return -1;
    }
    *v = (int64_t)PyLong_AsUnsignedLongLongMask(r);
    Py_DECREF(r);
  }
  return PyErr_Occurred() ? -1 : 0;
}

/* kinds: one letter per argument, t a tensor, i an integer (a size, an int32:
 * its low bits are taken), p an address as an int or None (NULL). */
static int values(PyObject* const* args, Py_ssize_t n, const char* kinds, int64_t* v) {
  for (Py_ssize_t i = 0; i < n; ++i) {
    if (!kinds[i]) break;
    if (kinds[i] == 't') {
      if (address(args[i], v + i)) return -1;
    } else if (kinds[i] == 'p' && args[i] == Py_None) {
      v[i] = 0;
    } else if (integer(args[i], v + i)) {
      return -1;
    }
  }
  return 0;
}

#define P(i) ((void*)(intptr_t)v[i])
#define ENTRY(name, kinds, call)                                                \
  static PyObject* name(PyObject* self, PyObject* const* args, Py_ssize_t na) { \
    int64_t v[sizeof(kinds) - 1];                                               \
    ifq_status st;                                                              \
    (void)self;                                                                 \
    if (na != (Py_ssize_t)sizeof(kinds) - 1)                                    \
      return PyErr_Format(PyExc_TypeError, "%zd arguments, %zd expected", na,   \
                          (Py_ssize_t)sizeof(kinds) - 1);                       \
    if (values(args, na, kinds, v)) return NULL;                                \
    Py_BEGIN_ALLOW_THREADS;                                                     \
    st = fn.call;                                                               \
    Py_END_ALLOW_THREADS;                                                       \
    return PyLong_FromLong(st);                                                 \
  }

ENTRY(conv_forward, "ptttp" "tttip",
      conv_forward(P(0), P(1), P(2), P(3), P(4), P(5), P(6), P(7), (size_t)v[8], P(9)))
ENTRY(conv_forward_fp4, "ptttptp", conv_forward_fp4(P(0), P(1), P(2), P(3), P(4), P(5), P(6)))
ENTRY(conv_pool_forward, "ppttttp", conv_pool_forward(P(0), P(1), P(2), P(3), P(4), P(5), P(6)))
ENTRY(conv_pool_forward_fp4, "ppttttp",
      conv_pool_forward_fp4(P(0), P(1), P(2), P(3), P(4), P(5), P(6)))
ENTRY(maxpool_codes, "pttp", maxpool_codes(P(0), P(1), P(2), P(3)))
ENTRY(convert_codes, "iiiiiittp",
      convert_codes(v[0], v[1], v[2], (int32_t)v[3], (int32_t)v[4], (int32_t)v[5], P(6), P(7),
                    P(8)))
ENTRY(run_stack, "ptttip", run_stack(P(0), P(1), P(2), P(3), (size_t)v[4], P(5)))
ENTRY(run_stack_static, "pttp", run_stack_static(P(0), P(1), P(2), P(3)))

/* bind(address, integer, addresses in the order of the table above) */
static PyObject* bind(PyObject* self, PyObject* const* args, Py_ssize_t na) {
  int64_t v[8];
  (void)self;
  if (na != 10) return PyErr_Format(PyExc_TypeError, "bind: 10 arguments expected");
  if (values(args + 2, 8, "pppppppp", v)) return NULL;
  Py_INCREF(args[0]);
  Py_XSETREF(conv_ptr, args[0]);
  Py_INCREF(args[1]);
  Py_XSETREF(conv_int, args[1]);
  fn.conv_forward = P(0);
  fn.conv_forward_fp4 = P(1);
  fn.conv_pool_forward = P(2);
  fn.conv_pool_forward_fp4 = P(3);
  fn.maxpool_codes = P(4);
  fn.convert_codes = P(5);
  fn.run_stack = P(6);
  fn.run_stack_static = P(7);
  Py_RETURN_NONE;
}

#define M(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, NULL}
static PyMethodDef methods[] = {M(bind), M(conv_forward), M(conv_forward_fp4),
                                M(conv_pool_forward), M(conv_pool_forward_fp4),
                                M(maxpool_codes), M(convert_codes), M(run_stack),
                                M(run_stack_static), {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ifqcall", NULL, -1, methods,
                                    NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__ifqcall(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  return s_data_ptr ? PyModule_Create(&module) : NULL;
}
