// Argument marshalling of the calls that a serving loop makes per layer and per step, as a CPython extension: a Caller holds the
// address of a C function and what kinds of arguments it takes, turns Python objects into pointers and numbers, calls it with
// the interpreter lock released, and returns its status.
//
// Through ctypes the marshalling of an attention call took 2.1 us (the launch itself takes 2.5), that of the description of a step of four
// requests 3.1; here they take 0.54 and 0.71.  Objects that are not met in such loops go to the Python functions that took all before.
#if !defined(__x86_64__) || defined(__ILP32__) || defined(_WIN32)
#error "arguments are passed as 64-bit integers, by the System V convention of x86-64"
#endif
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

enum { MAX_ARGS = 16, MAX_HELD = 8 };

// Kinds of arguments, one letter a Python argument:
//  S  structure of the registered type, by address      P  pointer: None, an address, or an object with data_ptr()
//  B  pointer, and behind it the object's nbytes        K  array of 32-bit integers; its length goes ahead of it
//  A  array of 32-bit integers                          i  32-bit integer
//  z  size                                              s  stream: None, a handle, or an object with cuda_stream
//  k, a  as K and A, but never copied: lists that the library reads once, or checks again as it uses them
typedef struct {
  PyObject_HEAD
  vectorcallfunc vectorcall;
  void* function;
  char kinds[MAX_ARGS];
  int n_kinds;
  PyObject* structure;     // type of S
  PyObject* address_of;    // Python: any object -> address or None
  PyObject* as_int32;      // Python: any object -> contiguous int32 array, or None
} Caller;

static PyObject *s_data_ptr, *s_nbytes, *s_cuda_stream;

// What a call holds on to until it is done: of each argument of kind S, K, A, k or a one thing, and caller_init sees to it that there are no more than MAX_HELD.
typedef struct {
  Py_buffer views[MAX_HELD];
  void* copies[MAX_HELD];
  int n, n_copies;
} Held;

static void release(Held* held) {
  while (held->n > 0) PyBuffer_Release(&held->views[--held->n]);
  while (held->n_copies > 0) PyMem_Free(held->copies[--held->n_copies]);
}

// Arrays of K and A of fewer bytes are copied while the interpreter lock is held: the library checks them and reads them again, and another thread
// may write to the caller's in between.  Larger ones are the caller's to leave alone during the call.  (The copies of the lengths of a step of four
// requests take 0.03 us of 0.71.  Two lists of 1514 page ids, copied, took 1.2 of the 21 us of a page copy: k and a.)
enum { COPY_BELOW = 1 << 14 };

static int integer(PyObject* o, uint64_t* out) {
  if (PyLong_Check(o)) {
    *out = PyLong_AsUnsignedLongLongMask(o);
  } else {
    PyObject* l = PyNumber_Long(o);
    if (!l) return -1;
    *out = PyLong_AsUnsignedLongLongMask(l);
    Py_DECREF(l);
  }
  return PyErr_Occurred() ? -1 : 0;
}

// Address as a Python object, which is consumed: an integer or None.
static int taken(PyObject* address, uint64_t* out) {
  int bad = !address;
  if (!bad) {
    *out = 0;
    if (address != Py_None) bad = integer(address, out);
    Py_DECREF(address);
  }
  return bad ? -1 : 0;
}

static int pointer(const Caller* self, PyObject* o, uint64_t* out) {
  if (o == Py_None) {
    *out = 0;
    return 0;
  }
  if (PyLong_Check(o)) return integer(o, out);
  PyObject* address = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!address) {
    if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return -1;
    PyErr_Clear();
    address = PyObject_CallOneArg(self->address_of, o);
  }
  return taken(address, out);
}

static int attribute(PyObject* o, PyObject* name, uint64_t* out) { return taken(PyObject_GetAttr(o, name), out); }

// The 32-bit integers of a one-dimensional array that lies as C does, without a copy.
static int plain_int32(PyObject* o, Py_buffer* view) {
  if (!PyObject_CheckBuffer(o)) return 0;
  if (PyObject_GetBuffer(o, view, PyBUF_ND | PyBUF_FORMAT) != 0) {      // refused where it is not contiguous
    PyErr_Clear();
    return 0;
  }
  if (view->ndim == 1 && view->itemsize == 4 && view->format && view->format[0] == 'i' && view->format[1] == 0) return 1;
  PyBuffer_Release(view);
  return 0;
}

static int int32_array(const Caller* self, PyObject* o, Held* held, uint64_t* address, uint64_t* length, int want_length, int copied) {
  Py_buffer* view = &held->views[held->n];
  if (plain_int32(o, view)) {
    *length = (uint64_t)view->shape[0];
  } else {
    PyObject* a = PyObject_CallOneArg(self->as_int32, o);
    if (!a) return -1;
    Py_ssize_t n = 0;
    int bad = 0;
    if (want_length) bad = (n = PyObject_Size(a)) < 0;                    // of None and of a single number: an error
    if (!bad && a == Py_None) {
      Py_DECREF(a);
      *address = 0;
      return 0;
    }
    if (!bad) bad = PyObject_GetBuffer(a, view, PyBUF_SIMPLE) != 0;       // (the view keeps the array alive)
    Py_DECREF(a);
    if (bad) return -1;
    *length = (uint64_t)n;
  }
  if (copied && view->len < COPY_BELOW) {
    void* copy = PyMem_Malloc((size_t)view->len);
    if (copy && view->len > 0) memcpy(copy, view->buf, (size_t)view->len);
    PyBuffer_Release(view);
    if (!copy) {
      PyErr_NoMemory();
      return -1;
    }
    held->copies[held->n_copies++] = copy;
    *address = (uint64_t)(uintptr_t)copy;
    return 0;
  }
  *address = (uint64_t)(uintptr_t)view->buf;
  held->n++;
  return 0;
}

typedef int32_t (*Function)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t);

static PyObject* call(PyObject* callable, PyObject* const* args, size_t nargsf, PyObject* kwnames) {
  const Caller* self = (const Caller*)callable;
  const Py_ssize_t n_args = PyVectorcall_NARGS(nargsf);
  if (!self->function || n_args != self->n_kinds || (kwnames && PyTuple_GET_SIZE(kwnames) != 0)) {
    PyErr_Format(PyExc_TypeError, "%d positional arguments are needed", self->n_kinds);
    return NULL;
  }
  uint64_t a[MAX_ARGS + 2] = {0};
  int n = 0, bad = 0;
  Held held;
  held.n = held.n_copies = 0;
  for (int i = 0; i < self->n_kinds && !bad; ++i) {
    PyObject* o = args[i];
    switch (self->kinds[i]) {
      case 'S':
        if (!PyObject_TypeCheck(o, (PyTypeObject*)self->structure)) {
          PyErr_Format(PyExc_TypeError, "a %s is needed, not a %s", ((PyTypeObject*)self->structure)->tp_name, Py_TYPE(o)->tp_name);
          bad = 1;
        } else {
          bad = PyObject_GetBuffer(o, &held.views[held.n], PyBUF_SIMPLE) != 0;
          if (!bad) a[n++] = (uint64_t)(uintptr_t)held.views[held.n++].buf;
        }
        break;
      case 'P':
        bad = pointer(self, o, &a[n++]) != 0;
        break;
      case 'B':
        bad = pointer(self, o, &a[n++]) != 0;
        if (!bad && o != Py_None) bad = attribute(o, s_nbytes, &a[n]) != 0;
        ++n;
        break;
      case 'K':
      case 'k': {
        uint64_t length = 0;
        bad = int32_array(self, o, &held, &a[n + 1], &length, 1, self->kinds[i] == 'K') != 0;
        a[n] = length;
        n += 2;
        break;
      }
      case 'A':
      case 'a': {
        uint64_t length = 0;
        bad = int32_array(self, o, &held, &a[n++], &length, 0, self->kinds[i] == 'A') != 0;
        break;
      }
      case 'i':
      case 'z':
        bad = integer(o, &a[n++]) != 0;
        break;
      default:      // 's'
        if (o == Py_None) a[n++] = 0;
        else bad = (PyLong_Check(o) ? integer(o, &a[n]) : attribute(o, s_cuda_stream, &a[n])) != 0, ++n;
    }
  }
  int32_t status = 0;
  if (!bad) {
    // Integers and pointers travel alike, in order, and a function takes no notice of what is behind its own (System V, x86-64).
    Py_BEGIN_ALLOW_THREADS
    status = ((Function)(uintptr_t)self->function)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11]);
    Py_END_ALLOW_THREADS
  }
  release(&held);
  return bad ? NULL : PyLong_FromLong(status);
}

static int caller_init(PyObject* o, PyObject* args, PyObject* kwargs) {
  Caller* self = (Caller*)o;
  unsigned long long address;
  const char* kinds;
  PyObject *structure, *address_of, *as_int32;
  if (kwargs && PyDict_GET_SIZE(kwargs) != 0) {
    PyErr_SetString(PyExc_TypeError, "no keywords");
    return -1;
  }
  if (!PyArg_ParseTuple(args, "KsO!OO", &address, &kinds, &PyType_Type, &structure, &address_of, &as_int32)) return -1;
  int n = 0, words = 0, held = 0;
  for (; kinds[n]; ++n) {
    if (n == MAX_ARGS || !strchr("SPBKAkaizs", kinds[n])) break;
    words += kinds[n] == 'B' || kinds[n] == 'K' || kinds[n] == 'k' ? 2 : 1;
    held += strchr("SKAka", kinds[n]) != NULL;
    self->kinds[n] = kinds[n];
  }
  if (kinds[n] || words > 12 || held > MAX_HELD || address == 0) {
    PyErr_SetString(PyExc_ValueError, "kinds of at most 12 arguments out of SPBKAkaizs, at most 8 of them SKAka, and an address");
    return -1;
  }
  self->n_kinds = n;
  self->function = (void*)(uintptr_t)address;
  self->vectorcall = call;
  Py_INCREF(structure);
  Py_XSETREF(self->structure, structure);
  Py_INCREF(address_of);
  Py_XSETREF(self->address_of, address_of);
  Py_INCREF(as_int32);
  Py_XSETREF(self->as_int32, as_int32);
  return 0;
}

static void caller_dealloc(PyObject* o) {
  Caller* self = (Caller*)o;
  Py_XDECREF(self->structure);
  Py_XDECREF(self->address_of);
  Py_XDECREF(self->as_int32);
  Py_TYPE(o)->tp_free(o);
}

static PyObject* caller_new(PyTypeObject* type, PyObject* args, PyObject* kwargs) {
  Caller* self = (Caller*)type->tp_alloc(type, 0);
  if (self) self->vectorcall = call;
  return (PyObject*)self;
}

static PyTypeObject caller_type = {
    PyVarObject_HEAD_INIT(NULL, 0).tp_name = "_hfxcall.Caller",
    .tp_basicsize = sizeof(Caller),
    .tp_dealloc = caller_dealloc,
    .tp_vectorcall_offset = offsetof(Caller, vectorcall),
    .tp_call = PyVectorcall_Call,
    .tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL,
    .tp_doc = "Caller(address, kinds, structure type, address_of, as_int32)",
    .tp_init = caller_init,
    .tp_new = caller_new,
};

static struct PyModuleDef module = {
    PyModuleDef_HEAD_INIT, .m_name = "_hfxcall", .m_doc = "Argument marshalling of libhfxattn's calls.", .m_size = -1};

PyMODINIT_FUNC PyInit__hfxcall(void) {
  if (!(s_data_ptr = PyUnicode_InternFromString("data_ptr")) || !(s_nbytes = PyUnicode_InternFromString("nbytes")) ||
      !(s_cuda_stream = PyUnicode_InternFromString("cuda_stream")) || PyType_Ready(&caller_type) < 0)
    return NULL;
  PyObject* m = PyModule_Create(&module);
  if (!m) return NULL;
  Py_INCREF(&caller_type);
  if (PyModule_AddObject(m, "Caller", (PyObject*)&caller_type) < 0) {
    Py_DECREF(&caller_type);
    Py_DECREF(m);
    return NULL;
  }
  return m;
}
