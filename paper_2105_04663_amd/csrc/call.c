/* The two Dot entry points called from Python without ctypes, for arguments in their plain form: descriptor objects whose C form the binding
 * holds (made from the very field objects they still have), lists or tuples of ShardBuf with int fields and of int fill counts.  Anything else is
 * handed back (None), and the binding converts it as ever, with the errors that belong to it.
 *
 * What a small call costs on the host is this conversion: of a Dot over 4 partitions 7.7 of 10.5 us, over 32 21 of 30 (ctypes, attribute by
 * attribute in Python); with it 0.9 and 4.
 */
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <stdint.h>
#include <string.h>

#include "../../include/gspmd.h"

typedef int32_t (*grouped_fn)(const gspmd_mesh*, const gspmd_dot_dims*, const gspmd_shard_buf*, const gspmd_sharding*, const gspmd_shard_buf*, const gspmd_sharding*,
                              const gspmd_shard_buf*, const gspmd_sharding*, const int64_t*, int32_t, void*, int64_t, void*);
typedef int32_t (*local_fn)(const gspmd_mesh*, const gspmd_dot_dims*, const gspmd_shard_buf*, const gspmd_sharding*, const gspmd_shard_buf*, const gspmd_sharding*,
                            const gspmd_shard_buf*, const gspmd_sharding*, int64_t, const int64_t*, int32_t, void*, int64_t, void*);

static grouped_fn grouped = NULL;
static local_fn local = NULL;
static PyObject *mesh_type, *dims_type, *sharding_type, *buf_type;
static PyObject *s_held, *s_data, *s_dtype, *s_row_stride;
static PyObject *mesh_fields[2], *sharding_fields[2], *dims_fields[4];

/* What `obj` holds its C form by, if its fields are the objects that it was made from; a new reference, since another thread may give the object
 * other fields while a call is under way. */
static PyObject* held_form(PyObject* obj, PyObject* type, PyObject** fields, Py_ssize_t n) {
  if ((PyObject*)Py_TYPE(obj) != type) return NULL;
  PyObject* dict = PyObject_GenericGetDict(obj, NULL);
  if (!dict) {
    PyErr_Clear();
    return NULL;
  }
  PyObject* held = PyDict_GetItem(dict, s_held);
  int same = held && PyTuple_CheckExact(held) && PyTuple_GET_SIZE(held) == 4;
  if (same) {
    PyObject* of = PyTuple_GET_ITEM(held, 0);
    same = PyTuple_CheckExact(of) && PyTuple_GET_SIZE(of) == n && PyLong_CheckExact(PyTuple_GET_ITEM(held, 3));
    for (Py_ssize_t i = 0; same && i < n; ++i) same = PyDict_GetItem(dict, fields[i]) == PyTuple_GET_ITEM(of, i);
  }
  if (same) Py_INCREF(held);
  Py_DECREF(dict);
  return same ? held : NULL;
}

/* the five descriptors of a Dot */
typedef struct {
  PyObject* held[5];
  const gspmd_mesh* mesh;
  const gspmd_dot_dims* dims;
  const gspmd_sharding *lhs, *rhs, *out;
} forms;
static void let_go(forms* f) {
  for (int i = 0; i < 5; ++i) Py_CLEAR(f->held[i]);
}
static int hold(PyObject* const* a, forms* f) {
  memset(f, 0, sizeof(*f));
  if (!(f->held[0] = held_form(a[0], mesh_type, mesh_fields, 2)) || !(f->held[1] = held_form(a[1], dims_type, dims_fields, 4)) ||
      !(f->held[2] = held_form(a[3], sharding_type, sharding_fields, 2)) || !(f->held[3] = held_form(a[5], sharding_type, sharding_fields, 2)) ||
      !(f->held[4] = held_form(a[7], sharding_type, sharding_fields, 2))) {
    let_go(f);
    return 0;
  }
  void* at[5];
  for (int i = 0; i < 5; ++i) at[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(f->held[i], 3));
  f->mesh = at[0]; f->dims = at[1]; f->lhs = at[2]; f->rhs = at[3]; f->out = at[4];
  return 1;
}

/* an int (no subclass, no bool) of 64 bits; 0 if it is not */
static int plain_int(PyObject* v, int64_t* out) {
  int overflow = 0;
  if (!v || !PyLong_CheckExact(v)) return 0;
  *out = PyLong_AsLongLongAndOverflow(v, &overflow);
  return !overflow;
}

static int shard(PyObject* obj, gspmd_shard_buf* out) {
  int64_t data, dtype, stride;
  if ((PyObject*)Py_TYPE(obj) != buf_type) return 0;
  PyObject* dict = PyObject_GenericGetDict(obj, NULL);
  if (!dict) {
    PyErr_Clear();
    return 0;
  }
  const int plain = plain_int(PyDict_GetItem(dict, s_data), &data) && plain_int(PyDict_GetItem(dict, s_dtype), &dtype) &&
                    plain_int(PyDict_GetItem(dict, s_row_stride), &stride) && data >= 0 && dtype == (int32_t)dtype;
  Py_DECREF(dict);
  if (!plain) return 0;
  memset(out, 0, sizeof(*out));
  out->data = (void*)(uintptr_t)data;
  out->dtype = (int32_t)dtype;
  out->row_stride = stride;
  return 1;
}

static int shards(PyObject* seq, int64_t n, gspmd_shard_buf* out) {
  if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return 0;
  if (PySequence_Fast_GET_SIZE(seq) != n) return 0;
  for (int64_t i = 0; i < n; ++i) {
    PyObject* item = PySequence_Fast_GET_ITEM(seq, i);
    if (i > 0 && item == PySequence_Fast_GET_ITEM(seq, i - 1)) out[i] = out[i - 1];       /* replicas share a buffer */
    else if (!shard(item, out + i)) return 0;
  }
  return 1;
}

/* Whether `n` fill counts are one for every entry of the lhs's batch dimensions at least: the library reads that many. */
static int enough_fills(const forms* f, Py_ssize_t n) {
  int64_t entries = 1;
  for (int32_t i = 0; i < f->dims->n_batch; ++i) {
    const int32_t d = f->dims->lhs_batch[i];
    if (d < 0 || d >= f->lhs->rank || f->lhs->global_shape[d] < 0) return 0;
    if (f->lhs->global_shape[d] > 0 && entries > n / f->lhs->global_shape[d]) return 0;
    entries *= f->lhs->global_shape[d];
  }
  return f->dims->n_batch >= 0 && entries <= n;
}

/* fill counts: none (*fill NULL), or a list or tuple of ints, in `few` or in memory of their own */
enum { kFills = 64 };
static int fills(PyObject* seq, const forms* f, int64_t* few, int64_t** fill) {
  *fill = NULL;
  if (seq == Py_None) return 1;
  if (!PyList_CheckExact(seq) && !PyTuple_CheckExact(seq)) return 0;
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
  if (n < 1 || !enough_fills(f, n) || !(*fill = n <= kFills ? few : PyMem_Malloc((size_t)n * sizeof(**fill)))) return 0;
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!plain_int(PySequence_Fast_GET_ITEM(seq, i), *fill + i)) {
      if (*fill != few) PyMem_Free(*fill);
      return 0;
    }
  return 1;
}

enum { kOnStack = 16, kMost = 1 << 20 };       /* partitions whose shards' C form is on the stack; of a mesh dimension */

/* grouped_dot(mesh, dims, lhs, lhs_sh, rhs, rhs_sh, out, out_sh, fill, epilogue, workspace, workspace_bytes, stream): status, or None */
static PyObject* grouped_dot(PyObject* self, PyObject* const* a, Py_ssize_t n_args) {
  (void)self;
  int64_t epilogue, workspace, bytes, stream, n = 1, few_fills[kFills], *fill;
  forms f;
  if (n_args != 13 || !grouped || !plain_int(a[9], &epilogue) || epilogue != (int32_t)epilogue || !plain_int(a[10], &workspace) || workspace < 0 ||
      !plain_int(a[11], &bytes) || !plain_int(a[12], &stream) || stream < 0 || !hold(a, &f)) Py_RETURN_NONE;
  for (int32_t i = 0; i < f.mesh->rank && n > 0; ++i) n = f.mesh->shape[i] < 1 || f.mesh->shape[i] > kMost || n > kMost ? 0 : n * f.mesh->shape[i];
  gspmd_shard_buf few[3 * kOnStack], *bufs = few;
  int plain = n > 0;
  if (plain && n > kOnStack) plain = (bufs = PyMem_Malloc((size_t)(3 * n) * sizeof(*bufs))) != NULL;
  plain = plain && shards(a[2], n, bufs) && shards(a[4], n, bufs + n) && shards(a[6], n, bufs + 2 * n) && fills(a[8], &f, few_fills, &fill);
  int32_t status = 0;
  if (plain) {
    Py_BEGIN_ALLOW_THREADS
    status = grouped(f.mesh, f.dims, bufs, f.lhs, bufs + n, f.rhs, bufs + 2 * n, f.out, fill, (int32_t)epilogue, (void*)(uintptr_t)workspace, bytes,
                     (void*)(uintptr_t)stream);
    Py_END_ALLOW_THREADS
    if (fill != few_fills) PyMem_Free(fill);
  }
  if (bufs != few) PyMem_Free(bufs);
  let_go(&f);
  if (!plain) Py_RETURN_NONE;
  return PyLong_FromLong(status);
}

/* local_dot(mesh, dims, lhs, lhs_sh, rhs, rhs_sh, out, out_sh, partition_id, fill, epilogue, workspace, workspace_bytes, stream): status, or None */
static PyObject* local_dot(PyObject* self, PyObject* const* a, Py_ssize_t n_args) {
  (void)self;
  int64_t pid, epilogue, workspace, bytes, stream, few_fills[kFills], *fill;
  gspmd_shard_buf l, r, o;
  forms f;
  if (n_args != 14 || !local || !plain_int(a[8], &pid) || !plain_int(a[10], &epilogue) || epilogue != (int32_t)epilogue || !plain_int(a[11], &workspace) ||
      workspace < 0 || !plain_int(a[12], &bytes) || !plain_int(a[13], &stream) || stream < 0 || !shard(a[2], &l) || !shard(a[4], &r) || !shard(a[6], &o) ||
      !hold(a, &f)) Py_RETURN_NONE;
  if (!fills(a[9], &f, few_fills, &fill)) {
    let_go(&f);
    Py_RETURN_NONE;
  }
  int32_t status;
  Py_BEGIN_ALLOW_THREADS
  status = local(f.mesh, f.dims, &l, f.lhs, &r, f.rhs, &o, f.out, pid, fill, (int32_t)epilogue, (void*)(uintptr_t)workspace, bytes, (void*)(uintptr_t)stream);
  Py_END_ALLOW_THREADS
  if (fill != few_fills) PyMem_Free(fill);
  let_go(&f);
  return PyLong_FromLong(status);
}

/* bind(address of gspmd_grouped_dot, of gspmd_local_dot, Mesh, DotDims, Sharding, ShardBuf) */
static PyObject* bind(PyObject* self, PyObject* args) {
  (void)self;
  PyObject *g, *l, *m, *d, *s, *b;
  if (!PyArg_ParseTuple(args, "OOOOOO", &g, &l, &m, &d, &s, &b)) return NULL;
  void *gp = PyLong_AsVoidPtr(g), *lp = PyLong_AsVoidPtr(l);
  if (PyErr_Occurred()) return NULL;
  Py_INCREF(m); Py_INCREF(d); Py_INCREF(s); Py_INCREF(b);       /* (for good: the binding's own classes) */
  mesh_type = m; dims_type = d; sharding_type = s; buf_type = b;
  memcpy(&grouped, &gp, sizeof(gp));
  memcpy(&local, &lp, sizeof(lp));
  Py_RETURN_NONE;
}

static PyMethodDef methods[] = {
  {"grouped_dot", (PyCFunction)(void (*)(void))grouped_dot, METH_FASTCALL, NULL},
  {"local_dot", (PyCFunction)(void (*)(void))local_dot, METH_FASTCALL, NULL},
  {"bind", bind, METH_VARARGS, NULL},
  {NULL, NULL, 0, NULL},
};
static struct PyModuleDef module = {PyModuleDef_HEAD_INIT, "_call", NULL, -1, methods, NULL, NULL, NULL, NULL};

PyMODINIT_FUNC PyInit__call(void) {
  s_held = PyUnicode_InternFromString("_held");
  s_data = PyUnicode_InternFromString("data");
  s_dtype = PyUnicode_InternFromString("dtype");
  s_row_stride = PyUnicode_InternFromString("row_stride");
  mesh_fields[0] = PyUnicode_InternFromString("shape");
  mesh_fields[1] = PyUnicode_InternFromString("device_ids");
  sharding_fields[0] = PyUnicode_InternFromString("global_shape");
  sharding_fields[1] = PyUnicode_InternFromString("dims_mapping");
  dims_fields[0] = PyUnicode_InternFromString("lhs_batch");
  dims_fields[1] = PyUnicode_InternFromString("rhs_batch");
  dims_fields[2] = PyUnicode_InternFromString("lhs_contract");
  dims_fields[3] = PyUnicode_InternFromString("rhs_contract");
  return PyModule_Create(&module);
}
