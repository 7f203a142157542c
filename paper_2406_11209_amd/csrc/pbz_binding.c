/* The calls of the Python binding that programs make over and over: tensors in, one C entry point called on torch's current stream.
 *
 * What it spares is the interpreter's share of a small call: with ctypes an operation on a 256 x 256 image took 4.4 (negate) to
 * 7.8 us (decompress) of host time, of which the entry point and its launch are some 3; now 3.7 to 5.1, and eleven of them in a row 51 us
 * instead of 68.  Nothing of torch's or of the library's
 * is linked: a tensor is asked for its address by the methods that Python code would use, and the entry points come as
 * addresses, so that several builds of the library can be loaded.  The interpreter lock is released around the entry point.
 *
 * Every function returns the entry point's status; -1000 never is one.  A tensor that is not a contiguous one on the device is
 * refused with ValueError before anything is called. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject *s_is_cuda, *s_is_contiguous, *s_data_ptr, *s_shape, *s_get_device;
static PyObject *get_device, *get_stream; /* of torch */

static int address_of(PyObject *t, void **out) {
  int cuda, contiguous;
  PyObject *v = PyObject_GetAttr(t, s_is_cuda);
  if (!v) return -1;
  cuda = PyObject_IsTrue(v);
  Py_DECREF(v);
  if (cuda < 0) return -1;
  contiguous = 0;
  if (cuda) {
    v = PyObject_CallMethodNoArgs(t, s_is_contiguous);
    if (!v) return -1;
    contiguous = PyObject_IsTrue(v);
    Py_DECREF(v);
    if (contiguous < 0) return -1;
  }
  if (!contiguous) {
    PyErr_SetString(PyExc_ValueError, "pbz takes contiguous device tensors");
    return -1;
  }
  v = PyObject_CallMethodNoArgs(t, s_data_ptr);
  if (!v) return -1;
  *out = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

static int optional_address_of(PyObject *t, void **out) {
  *out = NULL;
  return t == Py_None ? 0 : address_of(t, out);
}

/* t.shape[0] */
static int blocks_of(PyObject *t, int64_t *n) {
  PyObject *shape = PyObject_GetAttr(t, s_shape), *first;
  if (!shape) return -1;
  first = PySequence_GetItem(shape, 0);
  Py_DECREF(shape);
  if (!first) return -1;
  *n = PyLong_AsLongLong(first);
  Py_DECREF(first);
  return *n == -1 && PyErr_Occurred() ? -1 : 0;
}

/* torch's current stream on the current device; its number as an object, too, where the caller asks for that */
static int current_stream_object(void **out, PyObject **object) {
  PyObject *device, *stream;
  if (!get_device) {
    PyObject *c = PyImport_ImportModule("torch._C"), *d = NULL, *s = NULL;
    if (!c) return -1;
    d = PyObject_GetAttrString(c, "_cuda_getDevice");
    s = d ? PyObject_GetAttrString(c, "_cuda_getCurrentRawStream") : NULL;
    Py_DECREF(c);
    if (!s) {
      Py_XDECREF(d);
      return -1;
    }
    get_stream = s;
    get_device = d;
  }
  device = PyObject_CallNoArgs(get_device);
  if (!device) return -1;
  stream = PyObject_CallOneArg(get_stream, device);
  Py_DECREF(device);
  if (!stream) return -1;
  *out = PyLong_AsVoidPtr(stream);
  if (*out == NULL && PyErr_Occurred()) {
    Py_DECREF(stream);
    return -1;
  }
  if (object) *object = stream;
  else Py_DECREF(stream);
  return 0;
}

static int current_stream(void **out) { return current_stream_object(out, NULL); }

/* spaces[(device of t, stream)] = (address, bytes): 1, and 0 where there is none yet */
static int space_of(PyObject *spaces, PyObject *t, PyObject *stream, void **ws, size_t *bytes) {
  PyObject *device = PyObject_CallMethodNoArgs(t, s_get_device), *key, *space;
  if (!device) return -1;
  key = PyTuple_Pack(2, device, stream);
  Py_DECREF(device);
  if (!key) return -1;
  space = PyDict_GetItemWithError(spaces, key); /* borrowed; spaces keeps it while the lock is held */
  Py_DECREF(key);
  if (!space) return PyErr_Occurred() ? -1 : 0;
  *ws = PyLong_AsVoidPtr(PyTuple_GET_ITEM(space, 0));
  *bytes = PyLong_AsSize_t(PyTuple_GET_ITEM(space, 1));
  return PyErr_Occurred() ? -1 : 1;
}

static int expect(Py_ssize_t got, Py_ssize_t least, Py_ssize_t most) {
  if (got >= least && got <= most) return 0;
  PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
  return -1;
}

static int as_pointer(PyObject *v, void **out) {
  *out = PyLong_AsVoidPtr(v);
  return *out == NULL && PyErr_Occurred() ? -1 : 0;
}

#define CALL(expression)                 \
  do {                                   \
    Py_BEGIN_ALLOW_THREADS               \
    status = (expression);               \
    Py_END_ALLOW_THREADS                 \
  } while (0)

enum { kMaxTensors = 6 };

/* blocks(entry, codec, tensor whose first extent is the number of blocks, tensors...):
 * entry(codec, blocks, addresses..., stream) */
static PyObject *blocks(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *p[kMaxTensors], *s;
  int64_t k;
  int status = -1000;
  const int count = (int)n - 3;
  (void)self;
  if (expect(n, 5, 3 + kMaxTensors) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec) || blocks_of(args[2], &k)) return NULL;
  for (int i = 0; i < count; ++i)
    if (address_of(args[3 + i], p + i)) return NULL;
  if (current_stream(&s)) return NULL;
  switch (count) {
    case 2: CALL(((int (*)(void *, int64_t, void *, void *, void *))fn)(codec, k, p[0], p[1], s)); break;
    case 3: CALL(((int (*)(void *, int64_t, void *, void *, void *, void *))fn)(codec, k, p[0], p[1], p[2], s)); break;
    case 5:
      CALL(((int (*)(void *, int64_t, void *, void *, void *, void *, void *, void *))fn)(codec, k, p[0], p[1], p[2], p[3], p[4], s));
      break;
    case 6:
      CALL(((int (*)(void *, int64_t, void *, void *, void *, void *, void *, void *, void *))fn)(codec, k, p[0], p[1], p[2], p[3], p[4],
                                                                                                  p[5], s));
      break;
    default: PyErr_SetString(PyExc_TypeError, "no entry point takes that many tensors"); return NULL;
  }
  return PyLong_FromLong(status);
}

/* reduce(entry, codec, workspaces by device and stream, tensor whose first extent is the number of blocks, tensors...):
 * entry(codec, blocks, addresses..., workspace, bytes, stream); None where the first tensor's device and the stream have no workspace */
static PyObject *reduce(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *ws, *p[5], *s;
  PyObject *stream;
  int64_t k;
  size_t bytes;
  int status = -1000, found;
  const int count = (int)n - 4;
  (void)self;
  if (expect(n, 7, 9) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec) || blocks_of(args[3], &k)) return NULL;
  for (int i = 0; i < count; ++i)
    if (address_of(args[4 + i], p + i)) return NULL;
  if (current_stream_object(&s, &stream)) return NULL;
  found = space_of(args[2], args[4], stream, &ws, &bytes);
  Py_DECREF(stream);
  if (found < 0) return NULL;
  if (!found) Py_RETURN_NONE;
  switch (count) {
    case 3:
      CALL(((int (*)(void *, int64_t, void *, void *, void *, void *, size_t, void *))fn)(codec, k, p[0], p[1], p[2], ws, bytes, s));
      break;
    case 5:
      CALL(((int (*)(void *, int64_t, void *, void *, void *, void *, void *, void *, size_t, void *))fn)(codec, k, p[0], p[1], p[2], p[3],
                                                                                                        p[4], ws, bytes, s));
      break;
    default: PyErr_SetString(PyExc_TypeError, "no entry point takes that many tensors"); return NULL;
  }
  return PyLong_FromLong(status);
}

/* scalar(entry, codec, x, N, F, N_out, F_out): entry(codec, blocks of F, N, F, x, N_out, F_out, stream) */
static PyObject *scalar(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *p[4], *s;
  int64_t k;
  int status = -1000;
  double x;
  (void)self;
  if (expect(n, 7, 7) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec)) return NULL;
  x = PyFloat_AsDouble(args[2]);
  if (x == -1.0 && PyErr_Occurred()) return NULL;
  if (blocks_of(args[4], &k)) return NULL;
  for (int i = 0; i < 4; ++i)
    if (address_of(args[3 + i], p + i)) return NULL;
  if (current_stream(&s)) return NULL;
  CALL(((int (*)(void *, int64_t, void *, void *, double, void *, void *, void *))fn)(codec, k, p[0], p[1], x, p[2], p[3], s));
  return PyLong_FromLong(status);
}

/* compress(entry, codec, x, type of x, buffer of its extents, N, F): entry(codec, x, type, extents, N, F, stream) */
static PyObject *compress(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *x, *N, *F, *s;
  Py_buffer shape;
  long type;
  int status = -1000;
  (void)self;
  if (expect(n, 7, 7) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec) || address_of(args[2], &x)) return NULL;
  type = PyLong_AsLong(args[3]);
  if (type == -1 && PyErr_Occurred()) return NULL;
  if (address_of(args[5], &N) || address_of(args[6], &F) || current_stream(&s)) return NULL;
  if (PyObject_GetBuffer(args[4], &shape, PyBUF_SIMPLE)) return NULL;
  CALL(((int (*)(void *, void *, int, void *, void *, void *, void *))fn)(codec, x, (int)type, shape.buf, N, F, s));
  PyBuffer_Release(&shape);
  return PyLong_FromLong(status);
}

/* decompress(entry, codec, N, F, buffer of the extents, y, type of y): entry(codec, N, F, extents, y, type, stream) */
static PyObject *decompress(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *y, *N, *F, *s;
  Py_buffer shape;
  long type;
  int status = -1000;
  (void)self;
  if (expect(n, 7, 7) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec) || address_of(args[2], &N) || address_of(args[3], &F) ||
      address_of(args[5], &y))
    return NULL;
  type = PyLong_AsLong(args[6]);
  if (type == -1 && PyErr_Occurred()) return NULL;
  if (current_stream(&s)) return NULL;
  if (PyObject_GetBuffer(args[4], &shape, PyBUF_SIMPLE)) return NULL;
  CALL(((int (*)(void *, void *, void *, void *, void *, int, void *))fn)(codec, N, F, shape.buf, y, (int)type, s));
  PyBuffer_Release(&shape);
  return PyLong_FromLong(status);
}

/* segmented(entry, codec, workspaces, statistic, segments, blocks per segment, N1, F1, N2 or None, F2 or None, out): as reduce */
static PyObject *segmented(PyObject *self, PyObject *const *args, Py_ssize_t n) {
  void *fn, *codec, *ws, *p[5], *s;
  PyObject *stream;
  long what;
  int64_t segments, per;
  size_t bytes;
  int status = -1000, found;
  (void)self;
  if (expect(n, 11, 11) || as_pointer(args[0], &fn) || as_pointer(args[1], &codec)) return NULL;
  what = PyLong_AsLong(args[3]);
  segments = PyLong_AsLongLong(args[4]);
  per = PyLong_AsLongLong(args[5]);
  if ((what == -1 || segments == -1 || per == -1) && PyErr_Occurred()) return NULL;
  if (address_of(args[6], p) || address_of(args[7], p + 1) || optional_address_of(args[8], p + 2) || optional_address_of(args[9], p + 3) ||
      address_of(args[10], p + 4) || current_stream_object(&s, &stream))
    return NULL;
  found = space_of(args[2], args[6], stream, &ws, &bytes);
  Py_DECREF(stream);
  if (found < 0) return NULL;
  if (!found) Py_RETURN_NONE;
  CALL(((int (*)(void *, int, int64_t, int64_t, void *, void *, void *, void *, void *, void *, size_t, void *))fn)(
      codec, (int)what, segments, per, p[0], p[1], p[2], p[3], p[4], ws, bytes, s));
  return PyLong_FromLong(status);
}

static PyMethodDef methods[] = {{"blocks", (PyCFunction)(void (*)(void))blocks, METH_FASTCALL, NULL},
                                {"reduce", (PyCFunction)(void (*)(void))reduce, METH_FASTCALL, NULL},
                                {"scalar", (PyCFunction)(void (*)(void))scalar, METH_FASTCALL, NULL},
                                {"compress", (PyCFunction)(void (*)(void))compress, METH_FASTCALL, NULL},
                                {"decompress", (PyCFunction)(void (*)(void))decompress, METH_FASTCALL, NULL},
                                {"segmented", (PyCFunction)(void (*)(void))segmented, METH_FASTCALL, NULL},
                                {NULL, NULL, 0, NULL}};

static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__binding(void) {
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_shape = PyUnicode_InternFromString("shape");
  s_get_device = PyUnicode_InternFromString("get_device");
  if (!s_is_cuda || !s_is_contiguous || !s_data_ptr || !s_shape || !s_get_device) return NULL;
  return PyModule_Create(&module);
}
