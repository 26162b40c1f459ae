/* Calls of libbitdecode.so from Python without ctypes' conversion of every argument: the cache classes' steps and prefills.
 *
 * A step of a short context is bound by what the host does for it.  On a slow core KVCache.decode_step without the library's
 * own work 7.5 -> 2.7 us, PagedKVCache.quant_pack_kv 4.9 -> 2.7; issued one by one 8 paged prompts of up to 1333 tokens 43.7 ->
 * 39.7 us, a step of 6K tokens 9.3 -> 8.1.  Functions get the address of the library's entry point first (the library stays the one that
 * ctypes has loaded), a bd_cache / bd_paged_cache next (read through the buffer protocol), tensors as they are (their
 * data_ptr(); None is NULL), and return what the entry point returns.  As with ctypes, the interpreter's lock is released
 * during the call and integers are taken modulo 2^32.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>

static PyObject* name_data_ptr;

/* Address of a tensor's data, NULL for None; -1 with an exception set. */
static int tensor_address(PyObject* t, void** p) {
  *p = NULL;
  if (t == Py_None) return 0;
  PyObject* n = PyObject_CallMethodNoArgs(t, name_data_ptr);
  if (!n) return -1;
  *p = PyLong_AsVoidPtr(n);
  Py_DECREF(n);
  return !*p && PyErr_Occurred() ? -1 : 0;
}
static int address(PyObject* o, void** p) {
  *p = o == Py_None ? NULL : PyLong_AsVoidPtr(o);
  return !*p && PyErr_Occurred() ? -1 : 0;
}
static int int32_of(PyObject* o, int32_t* v) {
  const unsigned long n = PyLong_AsUnsignedLongMask(o);
  *v = (int32_t)(uint32_t)n;
  return n == (unsigned long)-1 && PyErr_Occurred() ? -1 : 0;
}
static int float_of(PyObject* o, float* v) {
  const double x = PyFloat_AsDouble(o);
  *v = (float)x;
  return x == -1.0 && PyErr_Occurred() ? -1 : 0;
}
/* A ctypes structure, which the caller's frame keeps alive. */
static int structure(PyObject* o, Py_buffer* b) { return PyObject_GetBuffer(o, b, PyBUF_SIMPLE); }
static int count_is(Py_ssize_t n, Py_ssize_t want) {
  if (n == want) return 1;
  PyErr_Format(PyExc_TypeError, "%zd arguments for %zd", n, want);
  return 0;
}

/* splits(fn, cache, packed_len) -> count   (bd_choose_splits, bd_step_splits) */
static PyObject* splits(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void* fn;
  int32_t len, count;
  Py_buffer c;
  (void)self;
  if (!count_is(n, 3) || address(a[0], &fn) || int32_of(a[2], &len) || structure(a[1], &c)) return NULL;
  count = ((int32_t(*)(const void*, int32_t))fn)(c.buf, len);
  PyBuffer_Release(&c);
  return PyLong_FromLong(count);
}

/* step(fn, cache, k_new, v_new, q, packed_len, res_len, scale, num_splits, workspace, out, stream)
 *   -> (status, packed_len, res_len)   (bd_decode_step, bd_decode_step_lazy) */
static PyObject* step(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void *fn, *k, *v, *q, *ws, *out, *stream;
  int32_t packed, res, ns;
  float scale;
  int status;
  Py_buffer c;
  (void)self;
  if (!count_is(n, 12) || address(a[0], &fn) || tensor_address(a[2], &k) || tensor_address(a[3], &v) || tensor_address(a[4], &q) ||
      int32_of(a[5], &packed) || int32_of(a[6], &res) || float_of(a[7], &scale) || int32_of(a[8], &ns) ||
      tensor_address(a[9], &ws) || tensor_address(a[10], &out) || address(a[11], &stream) || structure(a[1], &c))
    return NULL;
  Py_BEGIN_ALLOW_THREADS
  status = ((int (*)(const void*, const void*, const void*, const void*, int32_t*, int32_t*, float, int32_t, void*, void*,
                     void*))fn)(c.buf, k, v, q, &packed, &res, scale, ns, ws, out, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&c);
  return Py_BuildValue("(iii)", status, (int)packed, (int)res);
}

/* paged_step(fn, cache, k_new, v_new, q, scale, num_splits, workspace, out, stream) -> status
 *   (bd_paged_decode_step, bd_paged_counted_step and their lazy forms) */
static PyObject* paged_step(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void *fn, *k, *v, *q, *ws, *out, *stream;
  int32_t ns;
  float scale;
  int status;
  Py_buffer c;
  (void)self;
  if (!count_is(n, 10) || address(a[0], &fn) || tensor_address(a[2], &k) || tensor_address(a[3], &v) || tensor_address(a[4], &q) ||
      float_of(a[5], &scale) || int32_of(a[6], &ns) || tensor_address(a[7], &ws) || tensor_address(a[8], &out) ||
      address(a[9], &stream) || structure(a[1], &c))
    return NULL;
  Py_BEGIN_ALLOW_THREADS
  status = ((int (*)(const void*, const void*, const void*, const void*, float, int32_t, void*, void*, void*))fn)(
      c.buf, k, v, q, scale, ns, ws, out, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&c);
  return PyLong_FromLong(status);
}

/* paged_quant(fn, cache, seq, k, v, L, stream) -> status   (bd_paged_quant_pack_kv) */
static PyObject* paged_quant(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void *fn, *k, *v, *stream;
  int32_t seq, len;
  int status;
  Py_buffer c;
  (void)self;
  if (!count_is(n, 7) || address(a[0], &fn) || int32_of(a[2], &seq) || tensor_address(a[3], &k) || tensor_address(a[4], &v) ||
      int32_of(a[5], &len) || address(a[6], &stream) || structure(a[1], &c))
    return NULL;
  Py_BEGIN_ALLOW_THREADS
  status = ((int (*)(const void*, int32_t, const void*, const void*, int32_t, void*))fn)(c.buf, seq, k, v, len, stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&c);
  return PyLong_FromLong(status);
}

/* quant(fn, cache, k, v, L, stream) -> (status, packed_len, res_len)   (bd_quant_pack_kv) */
static PyObject* quant(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  void *fn, *k, *v, *stream;
  int32_t len, packed = 0, res = 0;
  int status;
  Py_buffer c;
  (void)self;
  if (!count_is(n, 6) || address(a[0], &fn) || tensor_address(a[2], &k) || tensor_address(a[3], &v) || int32_of(a[4], &len) ||
      address(a[5], &stream) || structure(a[1], &c))
    return NULL;
  Py_BEGIN_ALLOW_THREADS
  status = ((int (*)(const void*, const void*, const void*, int32_t, int32_t*, int32_t*, void*))fn)(c.buf, k, v, len, &packed, &res,
                                                                                                    stream);
  Py_END_ALLOW_THREADS
  PyBuffer_Release(&c);
  return Py_BuildValue("(iii)", status, (int)packed, (int)res);
}

static PyMethodDef methods[] = {
    {"splits", (PyCFunction)(void (*)(void))splits, METH_FASTCALL, NULL},
    {"step", (PyCFunction)(void (*)(void))step, METH_FASTCALL, NULL},
    {"paged_step", (PyCFunction)(void (*)(void))paged_step, METH_FASTCALL, NULL},
    {"paged_quant", (PyCFunction)(void (*)(void))paged_quant, METH_FASTCALL, NULL},
    {"quant", (PyCFunction)(void (*)(void))quant, METH_FASTCALL, NULL},
    {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_bdcall", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__bdcall(void) {
  name_data_ptr = PyUnicode_InternFromString("data_ptr");
  return name_data_ptr ? PyModule_Create(&module) : NULL;
}
