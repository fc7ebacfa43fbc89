// The calls that a training step or a served request makes (products, gradients, packing) from Python without ctypes: six functions
// of the binding's names and arguments that pass whole numbers straight to the library.  A small product is a launch, some 3.5 us of the
// host's time in the HIP runtime; ctypes' conversion of eleven arguments took 0.63 us of a call (1.38 on a slower processor) and takes 0.08
// (0.18) here.  The smallest product among others, both ways in turn in one process: 4.2 -> 3.8 us.
//
// Whatever is not the plain case -- keywords, other types than int and the binding's Mask, numbers out of range, a library not loaded yet,
// an error code -- goes to the binding's ctypes function of the same name, so that every call is accepted, refused and reported as there.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

typedef int (*pack_fn)(void *, int, void *, void *, void *);
typedef int (*spmm_fn)(void *, int, int64_t, int64_t, int64_t, void *, void *, int64_t, void *, int64_t, void *);
typedef int (*sddmm_fn)(void *, int, int64_t, int64_t, int64_t, void *, int64_t, void *, int64_t, void *, void *);
typedef int (*conv_fn)(void *, int, int64_t, int64_t, int64_t, int64_t, int64_t, void *, void *, void *, int64_t, void *);
typedef int (*conv_sddmm_fn)(void *, int, int64_t, int64_t, int64_t, int64_t, int64_t, void *, int64_t, void *, void *, void *);

enum { PACK, PACK_T, SPMM, SDDMM, CONV, CONV_SDDMM, COUNT };
// arguments after the mask: i dtype, q 64-bit number, p address; the last one (the stream) may be left out
static const char *const kinds[COUNT] = {"ippp", "ippp", "iqqqppqpqp", "iqqqpqpqpp", "iqqqqqpppqp", "iqqqqqpqppp"};
static void *address[COUNT];   // of the library's functions; NULL: not loaded
static PyObject *slow[COUNT];  // the binding's ctypes functions
static PyObject *mask_type, *pointer_type, *check, *str_handle, *str_value;

typedef union {
  int64_t q;
  void *p;
} Arg;

// 1: taken, 0: not the plain case (no Python error is left)
static int number(PyObject *o, char kind, Arg *a) {
  if (!PyLong_CheckExact(o)) return 0;
  int overflow;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) return 0;   // (an address above 2^63 is no user's)
  if (kind == 'i' ? v != (int)v : kind == 'p' ? v < 0 : 0) return 0;
  if (kind == 'p') a->p = (void *)(uintptr_t)v;
  else a->q = v;
  return 1;
}

static int mask_handle(PyObject *mask, void **out) {
  if ((PyObject *)Py_TYPE(mask) != mask_type) return 0;
  PyObject *handle = PyObject_GetAttr(mask, str_handle);
  int taken = 0;
  if (handle && (PyObject *)Py_TYPE(handle) == pointer_type) {
    PyObject *value = PyObject_GetAttr(handle, str_value);
    if (value && PyLong_CheckExact(value)) {
      *out = PyLong_AsVoidPtr(value);
      taken = *out != NULL;
    }
    Py_XDECREF(value);
  }
  Py_XDECREF(handle);
  if (!taken) PyErr_Clear();
  return taken;
}

static PyObject *call(int which, PyObject *const *args, Py_ssize_t n, PyObject *kwnames) {
  const char *kind = kinds[which];
  const Py_ssize_t most = (Py_ssize_t)strlen(kind) + 1;
  Arg a[12] = {{0}};
  void *m;
  int plain = address[which] && !(kwnames && PyTuple_GET_SIZE(kwnames)) && (n == most || n == most - 1) && mask_handle(args[0], &m);
  for (Py_ssize_t k = 1; plain && k < n; ++k) plain = number(args[k], kind[k - 1], &a[k]);
  if (!plain) {
    if (!slow[which]) {
      PyErr_SetString(PyExc_RuntimeError, "the binding has not been set up");
      return NULL;
    }
    return PyObject_Vectorcall(slow[which], args, (size_t)n, kwnames);
  }
  const int dt = (int)a[1].q;
  void *const f = address[which];
  int rc = 0;
  // (a launch, and in a mask's first call memory and tables: other threads may run, as under ctypes)
  Py_BEGIN_ALLOW_THREADS
  switch (which) {
    case PACK:
    case PACK_T: rc = ((pack_fn)f)(m, dt, a[2].p, a[3].p, a[4].p); break;
    case SPMM: rc = ((spmm_fn)f)(m, dt, a[2].q, a[3].q, a[4].q, a[5].p, a[6].p, a[7].q, a[8].p, a[9].q, a[10].p); break;
    case SDDMM: rc = ((sddmm_fn)f)(m, dt, a[2].q, a[3].q, a[4].q, a[5].p, a[6].q, a[7].p, a[8].q, a[9].p, a[10].p); break;
    case CONV: rc = ((conv_fn)f)(m, dt, a[2].q, a[3].q, a[4].q, a[5].q, a[6].q, a[7].p, a[8].p, a[9].p, a[10].q, a[11].p); break;
    case CONV_SDDMM: rc = ((conv_sddmm_fn)f)(m, dt, a[2].q, a[3].q, a[4].q, a[5].q, a[6].q, a[7].p, a[8].q, a[9].p, a[10].p, a[11].p); break;
  }
  Py_END_ALLOW_THREADS
  if (!rc) Py_RETURN_NONE;
  static const char *const names[COUNT] = {"rbgp_pack_device", "rbgp_pack_transposed_device", "rbgp_spmm", "rbgp_sddmm", "rbgp_conv3x3",
                                           "rbgp_conv3x3_sddmm"};
  return PyObject_CallFunction(check, "is", rc, names[which]);   // (raises)
}

#define FUNCTION(name, which) \
  static PyObject *name(PyObject *self, PyObject *const *args, Py_ssize_t n, PyObject *kw) { return call(which, args, n, kw); }
FUNCTION(pack_device, PACK)
FUNCTION(pack_transposed_device, PACK_T)
FUNCTION(spmm, SPMM)
FUNCTION(sddmm, SDDMM)
FUNCTION(conv3x3, CONV)
FUNCTION(conv3x3_sddmm, CONV_SDDMM)

// setup(Mask, c_void_p, _check, the six ctypes functions in the order of the enum)
static PyObject *setup(PyObject *self, PyObject *args) {
  PyObject *o[3 + COUNT];
  if (!PyArg_ParseTuple(args, "OOOOOOOOO", &o[0], &o[1], &o[2], &o[3], &o[4], &o[5], &o[6], &o[7], &o[8])) return NULL;
  for (int k = 0; k < 3 + COUNT; ++k) {
    PyObject **to = k == 0 ? &mask_type : k == 1 ? &pointer_type : k == 2 ? &check : &slow[k - 3];
    Py_INCREF(o[k]);
    Py_XSETREF(*to, o[k]);
  }
  Py_RETURN_NONE;
}

// loaded(six addresses)
static PyObject *loaded(PyObject *self, PyObject *args) {
  unsigned long long v[COUNT];
  if (!PyArg_ParseTuple(args, "KKKKKK", &v[0], &v[1], &v[2], &v[3], &v[4], &v[5])) return NULL;
  for (int k = 0; k < COUNT; ++k) address[k] = (void *)(uintptr_t)v[k];
  Py_RETURN_NONE;
}

#define FAST(name, fn, signature) {name, (PyCFunction)(void (*)(void))fn, METH_FASTCALL | METH_KEYWORDS, name signature "\n--\n\n"}
static PyMethodDef methods[] = {
    FAST("rbgp_pack_device", pack_device, "(mask, dtype, dev_values_ptr, dev_packed_ptr, stream=0)"),
    FAST("rbgp_pack_transposed_device", pack_transposed_device, "(mask_t, dtype, dev_values_ptr, dev_packed_ptr, stream=0)"),
    FAST("rbgp_spmm", spmm, "(mask, dtype, M, K, N, dev_packed_ptr, dev_I_ptr, ldI, dev_O_ptr, ldO, stream=0)"),
    FAST("rbgp_sddmm", sddmm, "(mask, dtype, M, K, N, dev_dO_ptr, ld_dO, dev_I_ptr, ldI, dev_dW_ptr, stream=0)"),
    FAST("rbgp_conv3x3", conv3x3,
         "(mask, dtype, channels_out, channels_in, images, height, width, dev_packed_ptr, dev_X_ptr, dev_O_ptr, ldO, stream=0)"),
    FAST("rbgp_conv3x3_sddmm", conv3x3_sddmm,
         "(mask, dtype, channels_out, channels_in, images, height, width, dev_dO_ptr, ld_dO, dev_X_ptr, dev_dW_ptr, stream=0)"),
    {"setup", setup, METH_VARARGS, NULL},
    {"loaded", loaded, METH_VARARGS, NULL},
    {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void) {
  str_handle = PyUnicode_InternFromString("handle");
  str_value = PyUnicode_InternFromString("value");
  if (!str_handle || !str_value) return NULL;
  return PyModule_Create(&module);
}
