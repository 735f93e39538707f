/* The per-call marshalling of the Python binding, in C: Python objects to the arguments of a C-ABI
 * entry point of libmipgemm.so, and the call with the GIL released.
 *
 * A pass of a quantized network is a run of calls of a few microseconds of device time each, so
 * what a call costs on the host bounds it.  Converting sixteen arguments through ctypes and asking
 * torch for the current stream took 5.5 us of a call's 7.5; here they take under 1 us.
 *
 * call(name, *args) returns the entry point's result, or None where an argument is of a type
 * that it leaves to the ctypes path (which converts it or raises): integers, pointers as None,
 * integers or objects with data_ptr(), streams as None (the current one), integers or objects with
 * cuda_stream, floats as float or int.  Integers are cut to their C width, as ctypes does. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

typedef int64_t q;
typedef void *p;
typedef int (*gemm_fn)(q, q, q, p, q, int, p, q, int, p, q, int, int, p, size_t, p);
typedef int (*gemm_scaled_fn)(q, q, q, p, q, int, p, q, int, p, q, int, int, p, size_t, p, float);
typedef int (*batched_fn)(q, q, q, p, q, int, q, p, q, int, q, p, q, int, q, q, int, p, size_t, p);
typedef int (*packed_fn)(q, q, q, p, q, int, p, p, q, int, int, p, size_t, p);
typedef int (*conv_fn)(q, q, q, q, q, q, q, q, q, p, p, p, int, p, size_t, p);
typedef int (*conv_scaled_fn)(q, q, q, q, q, q, q, q, q, p, p, p, int, p, size_t, p, float);
typedef int (*conv_sums_fn)(q, q, q, q, q, q, q, q, q, p, p, p, int, p, size_t, p, p);
typedef int (*conv_scaled_sums_fn)(q, q, q, q, q, q, q, q, q, p, p, p, int, p, size_t, p, float, p);

enum { GEMM, GEMM_SCALED, BATCHED, PACKED, CONV, CONV_SCALED, CONV_SUMS, CONV_SCALED_SUMS, KINDS };

/* q int64, i int, p pointer, z size, s stream, f float: the arguments of each kind in order */
static const char *const kFormat[KINDS] = {
    "qqqpqipqipqiipzs",  "qqqpqipqipqiipzsf", "qqqpqiqpqiqpqiqqipzs", "qqqpqippqiipzs",
    "qqqqqqqqqpppipzs",  "qqqqqqqqqpppipzsf", "qqqqqqqqqpppipzsp",    "qqqqqqqqqpppipzsfp"};
#define MOST_ARGS 20

typedef union { q i; p ptr; float f; } value;

typedef struct { int kind; void *fn; } entry;

static PyObject *entries;            /* name -> capsule of an entry */
static PyObject *s_data_ptr, *s_cuda_stream;
static PyObject *current_device, *raw_stream;  /* callables: () -> device, device -> stream handle */

static int whole(PyObject *o, q *to) {
  if (!PyLong_Check(o)) return 0;
  *to = (q)PyLong_AsUnsignedLongLongMask(o);
  return 1;
}

static int pointer(PyObject *o, p *to) {
  q v = 0;
  if (o == Py_None) { *to = NULL; return 1; }
  if (!whole(o, &v)) {
    PyObject *r = PyObject_CallMethodNoArgs(o, s_data_ptr);
    const int ok = r && whole(r, &v);
    Py_XDECREF(r);
    if (!ok) return 0;
  }
  *to = (p)(uintptr_t)v;
  return 1;
}

static int stream(PyObject *o, p *to) {
  q v = 0;
  if (o == Py_None) {
    PyObject *device, *handle;
    int ok;
    if (!current_device) return 0;
    device = PyObject_CallNoArgs(current_device);
    if (!device) return 0;
    handle = PyObject_CallOneArg(raw_stream, device);
    Py_DECREF(device);
    ok = handle && whole(handle, &v);
    Py_XDECREF(handle);
    if (!ok) return 0;
  } else if (!whole(o, &v)) {
    PyObject *r = PyObject_GetAttr(o, s_cuda_stream);
    const int ok = r && whole(r, &v);
    Py_XDECREF(r);
    if (!ok) return 0;
  }
  *to = (p)(uintptr_t)v;
  return 1;
}

static int convert(char as, PyObject *o, value *to) {
  switch (as) {
    case 'q': case 'i': case 'z': return whole(o, &to->i);
    case 'p': return pointer(o, &to->ptr);
    case 's': return stream(o, &to->ptr);
    default:
      if (!PyFloat_Check(o) && !PyLong_Check(o)) return 0;
      to->f = (float)PyFloat_AsDouble(o);
      return !PyErr_Occurred();
  }
}

static PyObject *call(PyObject *self, PyObject *const *args, Py_ssize_t nargs) {
  PyObject *capsule;
  const entry *e;
  const char *format;
  value a[MOST_ARGS];
  int n, rc = 0;
  (void)self;
  if (nargs < 1) { PyErr_SetString(PyExc_TypeError, "call(name, *args)"); return NULL; }
  capsule = PyDict_GetItemWithError(entries, args[0]);
  if (!capsule) {
    if (PyErr_Occurred()) return NULL;
    Py_RETURN_NONE;
  }
  e = (const entry *)PyCapsule_GetPointer(capsule, NULL);
  if (!e) return NULL;
  format = kFormat[e->kind];
  for (n = 0; format[n]; ++n) {
    if (n + 1 >= nargs || !convert(format[n], args[n + 1], &a[n])) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
  }
  if (n + 1 != nargs) Py_RETURN_NONE;
#define Q(k) a[k].i
#define I(k) (int)a[k].i
#define P(k) a[k].ptr
#define Z(k) (size_t)a[k].i
#define F(k) a[k].f
#define GEMM_ARGS Q(0), Q(1), Q(2), P(3), Q(4), I(5), P(6), Q(7), I(8), P(9), Q(10), I(11), I(12), P(13), Z(14), P(15)
#define CONV_ARGS \
  Q(0), Q(1), Q(2), Q(3), Q(4), Q(5), Q(6), Q(7), Q(8), P(9), P(10), P(11), I(12), P(13), Z(14), P(15)
  Py_BEGIN_ALLOW_THREADS
  switch (e->kind) {
    case GEMM: rc = ((gemm_fn)e->fn)(GEMM_ARGS); break;
    case GEMM_SCALED: rc = ((gemm_scaled_fn)e->fn)(GEMM_ARGS, F(16)); break;
    case BATCHED:
      rc = ((batched_fn)e->fn)(Q(0), Q(1), Q(2), P(3), Q(4), I(5), Q(6), P(7), Q(8), I(9), Q(10), P(11), Q(12), I(13),
                               Q(14), Q(15), I(16), P(17), Z(18), P(19));
      break;
    case PACKED:
      rc = ((packed_fn)e->fn)(Q(0), Q(1), Q(2), P(3), Q(4), I(5), P(6), P(7), Q(8), I(9), I(10), P(11), Z(12), P(13));
      break;
    case CONV: rc = ((conv_fn)e->fn)(CONV_ARGS); break;
    case CONV_SCALED: rc = ((conv_scaled_fn)e->fn)(CONV_ARGS, F(16)); break;
    case CONV_SUMS: rc = ((conv_sums_fn)e->fn)(CONV_ARGS, P(16)); break;
    default: rc = ((conv_scaled_sums_fn)e->fn)(CONV_ARGS, F(16), P(17)); break;
  }
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

static void release_entry(PyObject *capsule) { PyMem_Free(PyCapsule_GetPointer(capsule, NULL)); }

/* register(name, format, address): `format` names the kind by its arguments */
static PyObject *register_entry(PyObject *self, PyObject *args) {
  PyObject *name, *capsule;
  const char *format;
  unsigned long long address;
  entry *e;
  int kind = 0, bad;
  (void)self;
  if (!PyArg_ParseTuple(args, "UsK", &name, &format, &address)) return NULL;
  while (kind < KINDS && strcmp(kFormat[kind], format)) ++kind;
  if (kind == KINDS || !address) { PyErr_SetString(PyExc_ValueError, "unknown kind of entry point"); return NULL; }
  e = (entry *)PyMem_Malloc(sizeof(entry));
  if (!e) return PyErr_NoMemory();
  e->kind = kind;
  e->fn = (void *)(uintptr_t)address;
  capsule = PyCapsule_New(e, NULL, release_entry);
  if (!capsule) { PyMem_Free(e); return NULL; }
  bad = PyDict_SetItem(entries, name, capsule);
  Py_DECREF(capsule);
  if (bad) return NULL;
  Py_RETURN_NONE;
}

/* stream_source(current_device, raw_stream): where None as a stream is looked up from now on; None, None:
 * no longer here */
static PyObject *stream_source(PyObject *self, PyObject *args) {
  PyObject *device, *handle, *old_device = current_device, *old_handle = raw_stream;
  (void)self;
  if (!PyArg_ParseTuple(args, "OO", &device, &handle)) return NULL;
  if (device == Py_None || handle == Py_None) device = handle = NULL;
  Py_XINCREF(device);
  Py_XINCREF(handle);
  raw_stream = handle;
  current_device = device;
  Py_XDECREF(old_device);
  Py_XDECREF(old_handle);
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
    {"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL, "call(name, *args) -> result, or None"},
    {"register", register_entry, METH_VARARGS, "register(name, format, address)"},
    {"stream_source", stream_source, METH_VARARGS, "stream_source(current_device, raw_stream)"},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void) {
  entries = PyDict_New();
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!entries || !s_data_ptr || !s_cuda_stream) return NULL;
  return PyModule_Create(&module);
}
