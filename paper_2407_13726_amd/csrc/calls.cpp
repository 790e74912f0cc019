// The binding's calls without ctypes: one object per entry point of the C library that checks a call's arguments, asks torch for the addresses and
// the current stream, or takes the given one's handle, and calls.  It serves the ordinary call -- Python's or numpy's integers, torch tensors of the entry's type on a HIP device or
// None -- and leaves every other one, and every complaint, to the Python code in dastac.py.
//
// Why: a small product takes the GPU 3 to 4 us; the host took 4.1 to 4.5 through ctypes and takes 3.3 to 3.6 here, of which the launch itself is two (band_spmv n=8192
// 4.3 -> 3.6 us a call, ttm_ut n=30 4.5 -> 3.7, pack and unpack of n=512 9.1 -> 7.7).
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stddef.h>
#include <stdint.h>
#include <string.h>

namespace {

constexpr int kMostArgs = 12;

struct Entry {
  PyObject_HEAD
  vectorcallfunc call;
  void *address;             // of the C function; null: not bound
  int count;                 // arguments before the stream
  char kind[kMostArgs + 1];  // 'i' a 64-bit integer, 'f' a float32 tensor, 'd' a float64 tensor
};

PyObject *tensor_type, *dtypes[2], *raw_stream, *get_device, *declined;
PyObject *name_is_cuda, *name_dtype, *name_data_ptr, *name_cuda_stream;

// The answer for a call that the Python code has to make: -1.
PyObject *decline() {
  PyErr_Clear();
  Py_INCREF(declined);
  return declined;
}

bool address_of(PyObject *t, PyObject *dtype, int64_t &out) {
  if (t == Py_None) {
    out = 0;
    return true;
  }
  if ((PyObject *)Py_TYPE(t) != tensor_type) return false;
  PyObject *v = PyObject_GetAttr(t, name_is_cuda);
  if (!v) return false;
  const bool cuda = v == Py_True;
  Py_DECREF(v);
  if (!cuda || !(v = PyObject_GetAttr(t, name_dtype))) return false;
  const bool same = v == dtype;
  Py_DECREF(v);
  if (!same || !(v = PyObject_CallMethodNoArgs(t, name_data_ptr))) return false;
  out = (int64_t)PyLong_AsUnsignedLongLong(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}

// A Python integer or what numpy has for one.
bool integer_of(PyObject *v, int64_t &out) {
  int over = 0;
  if (PyLong_CheckExact(v)) {
    out = PyLong_AsLongLongAndOverflow(v, &over);
    return !over;
  }
  if (PyLong_Check(v) || !PyIndex_Check(v)) return false;
  PyObject *whole = PyNumber_Index(v);
  if (!whole) return false;
  out = PyLong_AsLongLongAndOverflow(whole, &over);
  Py_DECREF(whole);
  return !over && !PyErr_Occurred();
}

// arguments 0.. of the C function, whose parameters are all 64-bit integers or pointers
int invoke(void *f, int n, const int64_t *a) {
  typedef int64_t I;
  switch (n) {
    case 3: return ((int (*)(I, I, I))f)(a[0], a[1], a[2]);
    case 4: return ((int (*)(I, I, I, I))f)(a[0], a[1], a[2], a[3]);
    case 5: return ((int (*)(I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4]);
    case 6: return ((int (*)(I, I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4], a[5]);
    case 7: return ((int (*)(I, I, I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6]);
    case 8: return ((int (*)(I, I, I, I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]);
    case 9: return ((int (*)(I, I, I, I, I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8]);
    case 10: return ((int (*)(I, I, I, I, I, I, I, I, I, I))f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9]);
  }
  return -1;
}

PyObject *entry_call(PyObject *self, PyObject *const *args, size_t nargsf, PyObject *kwnames) {
  const Entry *e = (const Entry *)self;
  if (!e->address || kwnames || PyVectorcall_NARGS(nargsf) != e->count + 1) return decline();
  int64_t a[kMostArgs + 1];
  bool tensors = false;  // (with one, torch has a device)
  for (int k = 0; k < e->count; ++k) {
    if (e->kind[k] == 'i') {
      if (!integer_of(args[k], a[k])) return decline();
    } else {
      if (!address_of(args[k], dtypes[e->kind[k] == 'd'], a[k])) return decline();
      tensors |= args[k] != Py_None;
    }
  }
  if (!tensors) return decline();
  PyObject *stream;
  if (args[e->count] == Py_None) {
    PyObject *device = PyObject_CallNoArgs(get_device);
    stream = device ? PyObject_CallOneArg(raw_stream, device) : NULL;
    Py_XDECREF(device);
  } else {
    stream = PyObject_GetAttr(args[e->count], name_cuda_stream);
  }
  if (!stream) return decline();
  if (!PyLong_CheckExact(stream)) {
    Py_DECREF(stream);
    return decline();
  }
  a[e->count] = (int64_t)PyLong_AsUnsignedLongLong(stream);
  Py_DECREF(stream);
  if (PyErr_Occurred()) return decline();
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = invoke(e->address, e->count + 1, a);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(status);
}

PyTypeObject entry_type = {PyVarObject_HEAD_INIT(NULL, 0)};

// entry(kinds): an entry that declines until bind() gives it an address
PyObject *new_entry(PyObject *, PyObject *arg) {
  Py_ssize_t n;
  const char *kind = PyUnicode_AsUTF8AndSize(arg, &n);
  if (!kind) return NULL;
  if (n < 2 || n > 9 || strspn(kind, "ifd") != (size_t)n) {
    PyErr_SetString(PyExc_ValueError, "kinds: two to nine of i, f and d");
    return NULL;
  }
  Entry *e = PyObject_New(Entry, &entry_type);
  if (!e) return NULL;
  e->call = entry_call, e->address = NULL, e->count = (int)n;
  strcpy(e->kind, kind);
  return (PyObject *)e;
}

// bind(entry, address); address 0 makes it decline
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *e;
  unsigned long long address;
  if (!PyArg_ParseTuple(args, "O!K", &entry_type, &e, &address)) return NULL;
  ((Entry *)e)->address = (void *)(uintptr_t)address;
  Py_RETURN_NONE;
}

// torch(Tensor, float32, float64, raw_stream, get_device): what entries ask torch with; before bind
PyObject *set_torch(PyObject *, PyObject *args) {
  PyObject *t, *f, *d, *r, *g;
  if (!PyArg_ParseTuple(args, "OOOOO", &t, &f, &d, &r, &g)) return NULL;
  Py_INCREF(t), Py_INCREF(f), Py_INCREF(d), Py_INCREF(r), Py_INCREF(g);  // kept for the life of the process
  tensor_type = t, dtypes[0] = f, dtypes[1] = d, raw_stream = r, get_device = g;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"entry", new_entry, METH_O, NULL}, {"bind", bind, METH_VARARGS, NULL}, {"torch", set_torch, METH_VARARGS, NULL}, {NULL, NULL, 0, NULL}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_calls", NULL, -1, methods, NULL, NULL, NULL, NULL};

}  // namespace

PyMODINIT_FUNC PyInit__calls(void) {
  entry_type.tp_name = "paper_2407_13726_amd._calls.Entry";
  entry_type.tp_basicsize = sizeof(Entry);
  entry_type.tp_flags = Py_TPFLAGS_DEFAULT | Py_TPFLAGS_HAVE_VECTORCALL;
  entry_type.tp_vectorcall_offset = offsetof(Entry, call);
  entry_type.tp_call = PyVectorcall_Call;
  if (PyType_Ready(&entry_type) < 0) return NULL;
  declined = PyLong_FromLong(-1);
  name_is_cuda = PyUnicode_InternFromString("is_cuda");
  name_dtype = PyUnicode_InternFromString("dtype");
  name_data_ptr = PyUnicode_InternFromString("data_ptr");
  name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!declined || !name_is_cuda || !name_dtype || !name_data_ptr || !name_cuda_stream) return NULL;
  return PyModule_Create(&module);
}
