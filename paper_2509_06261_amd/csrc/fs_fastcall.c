/* Native marshaling of the binding's device calls (CPython module _fsfast).
 *
 * A small call (a decode step of a few short sequences, the append of a few rows) is bound by the host: through ctypes the
 * Python side of one cost 3.5 - 5 us on top of the library's 3.3 - 5 (attribute and dtype checks, addresses, the current
 * stream as an object, fifteen argument conversions), and the GPU waited for it.  Here the same checks and conversions take
 * 0.5 us: append of 450 rows 8.2 -> 3.9 us a call, decode of eight sequences of up to 256 tokens 8.6 -> 6.4 (the kernel's time).
 *
 * Every function returns the library's status code, or None for arguments that are not what a serving program passes (plain
 * ints, torch.Tensor itself, the binding's own structures) or that the binding's checks refuse: the caller then takes the
 * ctypes path, which accepts, converts and refuses as it always did.  Nothing is kept between calls but what init() was
 * given: types, interned names and the library's entry points. */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <limits.h>
#include <stdint.h>
#include <string.h>

#include "fineserve.h"

enum { MAX_STRUCTS = 8 }; /* (FS_MAX batches and appends of a call) */

static struct {
  PyObject *tensor, *float16, *float32, *int32, *c_void_p, *batch, *append, *get_device, *get_stream;
  int (*kv_append)(fs_pool*, fs_model_t, int, const void*, const void*, int, const int32_t*, const int32_t*, const int32_t*, int, int64_t, void*);
  int (*kv_append_multi)(fs_pool*, const fs_append_t*, int, void*);
  int (*decode)(fs_pool*, fs_model_t, int, int, float, const void*, const int32_t*, const int32_t*, int, int, void*, float*, void*, uint64_t, void*);
  int (*decode_multi)(fs_pool*, const fs_batch_t*, int, void*, uint64_t, void*);
  int (*decode_step)(fs_pool*, const fs_append_t*, int, const fs_batch_t*, int, void*, uint64_t, void*);
} L;
static PyObject *s_data_ptr, *s_dtype, *s_is_contiguous, *s_numel, *s_element_size, *s_size, *s_one;

/* The helpers below return 1, 0 for "not the fast path's case", or -1 with an exception set. */
static int is_tensor(PyObject* o) { return (PyObject*)Py_TYPE(o) == L.tensor; }

static int method_int(PyObject* o, PyObject* name, int64_t* out) {
  PyObject* r = PyObject_CallMethodNoArgs(o, name);
  if (!r) return -1;
  *out = (int64_t)PyLong_AsLongLong(r);
  Py_DECREF(r);
  return *out == -1 && PyErr_Occurred() ? -1 : 1;
}
static int size1(PyObject* o, int64_t* out) { /* tensor.shape[1]; fewer dimensions: the other path raises */
  PyObject* r = PyObject_CallMethodOneArg(o, s_size, s_one);
  if (!r) {
    if (!PyErr_ExceptionMatches(PyExc_IndexError)) return -1;
    PyErr_Clear();
    return 0;
  }
  *out = (int64_t)PyLong_AsLongLong(r);
  Py_DECREF(r);
  return *out == -1 && PyErr_Occurred() ? -1 : 1;
}
static int address(PyObject* o, void** out) {
  PyObject* r;
  if (!is_tensor(o)) return 0;
  r = PyObject_CallMethodNoArgs(o, s_data_ptr);
  if (!r) return -1;
  *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLong(r);
  Py_DECREF(r);
  return PyErr_Occurred() ? -1 : 1;
}
static int address_or_none(PyObject* o, void** out) {
  *out = NULL;
  return o == Py_None ? 1 : address(o, out);
}
static int has_dtype(PyObject* o, PyObject* a, PyObject* b) { /* (torch's dtypes are single objects) */
  PyObject* d = PyObject_GetAttr(o, s_dtype);
  if (!d) return -1;
  Py_DECREF(d);
  return d == a || d == b;
}
static int contiguous(PyObject* o) {
  PyObject* r = PyObject_CallMethodNoArgs(o, s_is_contiguous);
  if (!r) return -1;
  Py_DECREF(r);
  return r == Py_True;
}
static int plain_int(PyObject* o, int* out) {
  int over;
  long v;
  if (!PyLong_CheckExact(o)) return 0;
  v = PyLong_AsLongAndOverflow(o, &over);
  if (over || v < INT_MIN || v > INT_MAX) return 0;
  *out = (int)v;
  return 1;
}
/* the bytes of a ctypes object of exactly this type */
static int bytes_of(PyObject* o, PyObject* type, void* out, size_t n) {
  Py_buffer b;
  if ((PyObject*)Py_TYPE(o) != type) return 0;
  if (PyObject_GetBuffer(o, &b, PyBUF_SIMPLE) < 0) {
    PyErr_Clear();
    return 0;
  }
  if ((size_t)b.len == n) memcpy(out, b.buf, n);
  PyBuffer_Release(&b);
  return (size_t)b.len == n;
}
static int structs(PyObject* list, PyObject* type, void* out, size_t size, int* n) {
  Py_ssize_t i, k;
  if (!PyList_CheckExact(list)) return 0;
  k = PyList_GET_SIZE(list);
  if (k > MAX_STRUCTS) return 0;
  for (i = 0; i < k; ++i)
    if (bytes_of(PyList_GET_ITEM(list, i), type, (char*)out + (size_t)i * size, size) != 1) return 0;
  *n = (int)k;
  return 1;
}
/* stream: None for torch's current one (its device's), else not the fast path's case */
static int stream_of(PyObject* o, void** out) {
  PyObject *d, *r;
  if (o != Py_None) return 0;
  d = PyObject_CallNoArgs(L.get_device);
  if (!d) return -1;
  r = PyObject_CallOneArg(L.get_stream, d);
  Py_DECREF(d);
  if (!r) return -1;
  *out = (void*)(uintptr_t)PyLong_AsUnsignedLongLong(r);
  Py_DECREF(r);
  return PyErr_Occurred() ? -1 : 1;
}
static int workspace(PyObject* o, void** out, uint64_t* bytes) {
  int64_t n = 0, e = 0;
  int ok = address(o, out);
  if (ok != 1) return ok;
  if ((ok = method_int(o, s_numel, &n)) != 1) return ok;
  if ((ok = method_int(o, s_element_size, &e)) != 1) return ok;
  *bytes = (uint64_t)(n * e);
  return 1;
}

#define TRY(x)                       \
  do {                               \
    const int ok_ = (x);             \
    if (ok_ < 0) return NULL;        \
    if (ok_ == 0) Py_RETURN_NONE;    \
  } while (0)
#define CALL(expr)              \
  do {                          \
    int rc_;                    \
    Py_BEGIN_ALLOW_THREADS      \
    rc_ = (expr);               \
    Py_END_ALLOW_THREADS        \
    return PyLong_FromLong(rc_); \
  } while (0)
#define ARGS(want) \
  if (!L.tensor || n != (want)) Py_RETURN_NONE

/* (pool, model, layer, k, v, seq_idx, pos, block_tables, stream) */
static PyObject* kv_append(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  fs_pool* pool;
  int model, layer, i, f32;
  void *p[5], *stream;
  int64_t blocks, tokens;
  (void)self;
  ARGS(9);
  TRY(bytes_of(a[0], L.c_void_p, &pool, sizeof pool));
  TRY(plain_int(a[1], &model));
  TRY(plain_int(a[2], &layer));
  for (i = 0; i < 5; ++i) TRY(is_tensor(a[3 + i]));
  f32 = has_dtype(a[3], L.float32, L.float32);
  if (f32 < 0) return NULL;
  TRY(has_dtype(a[3], L.float16, L.float32));
  TRY(has_dtype(a[4], f32 ? L.float32 : L.float16, f32 ? L.float32 : L.float16));
  TRY(contiguous(a[3]));
  TRY(contiguous(a[4]));
  TRY(contiguous(a[7]));
  for (i = 5; i < 8; ++i) TRY(has_dtype(a[i], L.int32, L.int32));
  for (i = 0; i < 5; ++i) TRY(address(a[3 + i], &p[i]));
  TRY(size1(a[7], &blocks));
  TRY(method_int(a[5], s_numel, &tokens));
  if (blocks > INT_MAX) Py_RETURN_NONE;
  TRY(stream_of(a[8], &stream));
  CALL(L.kv_append(pool, model, layer, p[0], p[1], f32 ? FS_SRC_FP32 : FS_SRC_FP16, p[2], p[3], p[4], (int)blocks, tokens, stream));
}

/* (pool, appends, stream) */
static PyObject* kv_append_multi(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  fs_pool* pool;
  fs_append_t ap[MAX_STRUCTS];
  int k;
  void* stream;
  (void)self;
  ARGS(3);
  TRY(bytes_of(a[0], L.c_void_p, &pool, sizeof pool));
  TRY(structs(a[1], L.append, ap, sizeof ap[0], &k));
  TRY(stream_of(a[2], &stream));
  CALL(L.kv_append_multi(pool, ap, k, stream));
}

/* (pool, model, layer, n_q_heads, sm_scale, q, block_tables, seq_lens, out, lse, workspace, stream) */
static PyObject* decode_attention(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  fs_pool* pool;
  int model, layer, heads;
  float scale;
  void *q, *tables, *lens, *out, *lse, *ws, *stream;
  uint64_t bytes;
  int64_t seqs, blocks;
  (void)self;
  ARGS(12);
  TRY(bytes_of(a[0], L.c_void_p, &pool, sizeof pool));
  TRY(plain_int(a[1], &model));
  TRY(plain_int(a[2], &layer));
  TRY(plain_int(a[3], &heads));
  if (!PyFloat_CheckExact(a[4])) Py_RETURN_NONE;
  scale = (float)PyFloat_AS_DOUBLE(a[4]);
  TRY(address(a[5], &q));
  TRY(address(a[6], &tables));
  TRY(address(a[7], &lens));
  TRY(method_int(a[7], s_numel, &seqs));
  TRY(size1(a[6], &blocks));
  if (seqs > INT_MAX || blocks > INT_MAX) Py_RETURN_NONE;
  TRY(address_or_none(a[8], &out));
  TRY(address_or_none(a[9], &lse));
  TRY(workspace(a[10], &ws, &bytes));
  TRY(stream_of(a[11], &stream));
  CALL(L.decode(pool, model, layer, heads, scale, q, tables, lens, (int)seqs, (int)blocks, out, lse, ws, bytes, stream));
}

/* (pool, batches, workspace, stream) */
static PyObject* decode_attention_multi(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  fs_pool* pool;
  fs_batch_t b[MAX_STRUCTS];
  int k;
  void *ws, *stream;
  uint64_t bytes;
  (void)self;
  ARGS(4);
  TRY(bytes_of(a[0], L.c_void_p, &pool, sizeof pool));
  TRY(structs(a[1], L.batch, b, sizeof b[0], &k));
  TRY(workspace(a[2], &ws, &bytes));
  TRY(stream_of(a[3], &stream));
  CALL(L.decode_multi(pool, b, k, ws, bytes, stream));
}

/* (pool, appends, batches, workspace, stream) */
static PyObject* decode_step_multi(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  fs_pool* pool;
  fs_append_t ap[MAX_STRUCTS];
  fs_batch_t b[MAX_STRUCTS];
  int ka, kb;
  void *ws, *stream;
  uint64_t bytes;
  (void)self;
  ARGS(5);
  TRY(bytes_of(a[0], L.c_void_p, &pool, sizeof pool));
  TRY(structs(a[1], L.append, ap, sizeof ap[0], &ka));
  TRY(structs(a[2], L.batch, b, sizeof b[0], &kb));
  TRY(workspace(a[3], &ws, &bytes));
  TRY(stream_of(a[4], &stream));
  CALL(L.decode_step(pool, ap, ka, b, kb, ws, bytes, stream));
}

/* init(Tensor, float16, float32, int32, c_void_p, fs_batch_t, fs_append_t, get_device, get_stream, addresses of the five
 * entry points in the order of L); init() forgets them: every call is answered None until the next one */
static PyObject* init(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  PyObject** const objs[9] = {&L.tensor, &L.float16, &L.float32, &L.int32, &L.c_void_p, &L.batch, &L.append, &L.get_device, &L.get_stream};
  void* fn[5];
  int i;
  (void)self;
  if (n == 0) {
    for (i = 0; i < 9; ++i) Py_CLEAR(*objs[i]);
    Py_RETURN_NONE;
  }
  if (n != 14) {
    PyErr_SetString(PyExc_TypeError, "init takes 14 arguments or none");
    return NULL;
  }
  for (i = 0; i < 5; ++i) {
    fn[i] = PyLong_AsVoidPtr(a[9 + i]);
    if (!fn[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point");
      return NULL;
    }
  }
  memcpy(&L.kv_append, &fn[0], sizeof fn[0]);
  memcpy(&L.kv_append_multi, &fn[1], sizeof fn[0]);
  memcpy(&L.decode, &fn[2], sizeof fn[0]);
  memcpy(&L.decode_multi, &fn[3], sizeof fn[0]);
  memcpy(&L.decode_step, &fn[4], sizeof fn[0]);
  for (i = 8; i >= 0; --i) { /* (Tensor last: the other functions look at it first) */
    Py_INCREF(a[i]);
    Py_XSETREF(*objs[i], a[i]);
  }
  Py_RETURN_NONE;
}

#define FAST(name, doc) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, doc}
static PyMethodDef methods[] = {FAST(init, "Types and entry points of the calls."),
                                FAST(kv_append, "fs_kv_append, or None."),
                                FAST(kv_append_multi, "fs_kv_append_multi, or None."),
                                FAST(decode_attention, "fs_decode_attention, or None."),
                                FAST(decode_attention_multi, "fs_decode_attention_multi, or None."),
                                FAST(decode_step_multi, "fs_decode_step_multi, or None."),
                                {NULL, NULL, 0, NULL}};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fsfast", "Native marshaling of the binding's device calls.", -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__fsfast(void) {
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_dtype = PyUnicode_InternFromString("dtype");
  s_is_contiguous = PyUnicode_InternFromString("is_contiguous");
  s_numel = PyUnicode_InternFromString("numel");
  s_element_size = PyUnicode_InternFromString("element_size");
  s_size = PyUnicode_InternFromString("size");
  s_one = PyLong_FromLong(1);
  if (!s_data_ptr || !s_dtype || !s_is_contiguous || !s_numel || !s_element_size || !s_size || !s_one) return NULL;
  return PyModule_Create(&module);
}
