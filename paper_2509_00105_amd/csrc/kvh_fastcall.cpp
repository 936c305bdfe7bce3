// The calls of binding.py that a program makes per chunk, without ctypes: the arguments of an ordinary call are read from the
// tensors, checked as binding.py checks them, and handed to the C ABI.  Anything else (another type than torch.Tensor, a host
// tensor, an int that is none or does not fit, shapes or strides that do not match) returns None, and binding.py goes its own
// way, which accepts or refuses it.  Nothing is kept from one call to the next.
//
// One 256-token chunk of 4 layers decoded into pages took 8.2 us a call, 5 of them in Python and ctypes; the launch takes 2.4.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cstdint>

#include "../../include/kvh.h"

namespace {

// Looked up once, when the module is imported.
PyObject *tensor_type, *dtype_f16, *dtype_bf16, *dtype_i32;  // torch's
PyObject *s_is_cuda, *s_dtype, *s_shape, *s_stride, *s_data_ptr, *s_numel, *s_cuda_stream;

// The functions of one loaded library, and torch's queries for the current stream.
struct Calls {
  PyObject_HEAD
  decltype(&kvh_encode) encode;
  decltype(&kvh_encode_batch) encode_batch;
  decltype(&kvh_decode) decode;
  decltype(&kvh_decode_batch) decode_batch;
  decltype(&kvh_encode_kept) encode_kept;
  decltype(&kvh_decode_kept) decode_kept;
  PyObject *current_device, *raw_stream;
};

// What one call has read so far.  A failed step leaves ok false; an error raised on the way is dropped, because the slow path
// meets the same one, but not what is no error of the call (an interrupt, an exit).
struct Reader {
  bool ok = true;

  bool is_true(PyObject* t, PyObject* name) {
    PyObject* r = PyObject_GetAttr(t, name);
    const bool yes = r == Py_True;
    Py_XDECREF(r);
    return yes;
  }
  bool device_tensor(PyObject* t) { return Py_TYPE(t) == reinterpret_cast<PyTypeObject*>(tensor_type) && is_true(t, s_is_cuda); }
  bool has_dtype(PyObject* t, PyObject* dtype) {
    PyObject* r = PyObject_GetAttr(t, s_dtype);
    const bool same = r == dtype;
    Py_XDECREF(r);
    return same;
  }
  int64_t int_method(PyObject* t, PyObject* name) {
    PyObject* r = PyObject_CallMethodNoArgs(t, name);
    int64_t v = 0;
    if (r == nullptr || !PyLong_CheckExact(r)) ok = false; else v = PyLong_AsLongLong(r);
    Py_XDECREF(r);
    if (PyErr_Occurred()) ok = false;
    return v;
  }
  void* pointer(PyObject* t) {
    PyObject* r = PyObject_CallMethodNoArgs(t, s_data_ptr);
    void* p = nullptr;
    if (r == nullptr || !PyLong_CheckExact(r)) ok = false; else p = PyLong_AsVoidPtr(r);
    Py_XDECREF(r);
    if (PyErr_Occurred()) ok = false;
    return p;
  }
  // A device tensor of any type.
  void* device(PyObject* t) {
    if (ok && !device_tensor(t)) ok = false;
    return ok ? pointer(t) : nullptr;
  }
  // None, or a device tensor of int32 with at least `least` elements.
  int32_t* words(PyObject* t, int64_t least) {
    if (!ok || t == Py_None) return nullptr;
    if (!device_tensor(t) || !has_dtype(t, dtype_i32) || (least > 0 && int_method(t, s_numel) < least)) ok = false;
    return ok ? static_cast<int32_t*>(pointer(t)) : nullptr;
  }
  int64_t wide(PyObject* o) {
    if (!PyLong_CheckExact(o)) {
      ok = false;
      return 0;
    }
    int overflow = 0;
    const int64_t v = PyLong_AsLongLongAndOverflow(o, &overflow);
    if (overflow != 0) ok = false;
    return v;
  }
  int narrow(PyObject* o) {
    const int64_t v = wide(o);
    if (v < INT32_MIN || v > INT32_MAX) ok = false;
    return (int)v;
  }
  int dims(PyObject* tuple, int64_t (&out)[4]) {
    if (tuple == nullptr || !PyTuple_Check(tuple) || PyTuple_GET_SIZE(tuple) > 4) {
      ok = false;
      return 0;
    }
    const int n = (int)PyTuple_GET_SIZE(tuple);
    for (int i = 0; i < n; ++i) out[i] = wide(PyTuple_GET_ITEM(tuple, i));
    return n;
  }
};

// K and V: device tensors [l][tokens][c], or [l][blocks][block][c] when paged, of one 16-bit type, equal in shape and strides.
struct View {
  kvh_kv_view v;
  kvh_dtype dt;
  int l, tokens, c;
};

View read_view(Reader& r, PyObject* k, PyObject* v, bool paged) {
  View out{};
  if (!r.ok || !r.device_tensor(k) || !r.device_tensor(v)) {
    r.ok = false;
    return out;
  }
  PyObject* dt = PyObject_GetAttr(k, s_dtype);
  Py_XDECREF(dt);  // torch keeps its types
  if ((dt != dtype_f16 && dt != dtype_bf16) || !r.has_dtype(v, dt)) {
    r.ok = false;
    return out;
  }
  int64_t size[2][4], stride[2][4];
  int n[2];
  PyObject* t[2] = {k, v};
  for (int i = 0; i < 2; ++i) {
    PyObject* sizes = PyObject_GetAttr(t[i], s_shape);
    n[i] = r.dims(sizes, size[i]);
    Py_XDECREF(sizes);
    PyObject* strides = PyObject_CallMethodNoArgs(t[i], s_stride);
    if (r.dims(strides, stride[i]) != n[i]) r.ok = false;
    Py_XDECREF(strides);
  }
  const int want = paged ? 4 : 3;
  if (!r.ok || n[0] != want || n[1] != want) {
    r.ok = false;
    return out;
  }
  for (int i = 0; i < want; ++i)
    if (size[0][i] != size[1][i] || stride[0][i] != stride[1][i] || size[0][i] > INT32_MAX) r.ok = false;
  if (stride[0][want - 1] != 1 || (paged && stride[0][1] != stride[0][2] * size[0][2])) r.ok = false;
  out.dt = dt == dtype_f16 ? KVH_F16 : KVH_BF16;
  out.l = (int)size[0][0];
  out.tokens = (int)size[0][1];
  out.c = (int)size[0][want - 1];
  out.v.layer_stride = stride[0][0];
  out.v.token_stride = stride[0][want - 2];
  if (r.ok) {
    out.v.k = r.pointer(k);
    out.v.v = r.pointer(v);
  }
  return out;
}

void* read_stream(Reader& r, Calls* self, PyObject* stream) {
  if (!r.ok) return nullptr;
  PyObject* p = nullptr;
  if (stream != Py_None) {
    p = PyObject_GetAttr(stream, s_cuda_stream);
  } else if (PyObject* dev = PyObject_CallNoArgs(self->current_device)) {
    p = PyObject_CallOneArg(self->raw_stream, dev);
    Py_DECREF(dev);
  }
  void* out = nullptr;
  if (p == nullptr || !PyLong_CheckExact(p)) r.ok = false; else out = PyLong_AsVoidPtr(p);
  Py_XDECREF(p);
  if (PyErr_Occurred()) r.ok = false;
  return out;
}

// The status of `call()`, made without the interpreter's lock as ctypes makes it, or None for binding.py to take over.
template <typename F>
PyObject* finish(const Reader& r, F&& call) {
  if (!r.ok) {
    if (PyErr_Occurred() != nullptr && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

#define KVH_ARGS(N)                                                      \
  Calls* self = reinterpret_cast<Calls*>(self_);                         \
  if (n_args != (N)) {                                                   \
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");       \
    return nullptr;                                                      \
  }                                                                      \
  Reader r

// encode(k, v, level, blob, n_tokens or None, stream)
PyObject* encode(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(6);
  const View kv = read_view(r, a[0], a[1], false);
  const int level = r.narrow(a[2]), n = a[4] == Py_None ? kv.tokens : r.narrow(a[4]);
  void* blob = r.device(a[3]);
  const int64_t cap = r.ok ? r.int_method(a[3], s_numel) : 0;
  void* stream = read_stream(r, self, a[5]);
  return finish(r, [&] { return self->encode(&kv.v, kv.dt, kv.l, n, kv.c, level, blob, (size_t)cap, stream); });
}

// encode_batch(items, n_items, max_tokens_per_item, k, v, stream)
PyObject* encode_batch(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(6);
  const View kv = read_view(r, a[3], a[4], false);
  const void* items = r.device(a[0]);
  const int n = r.narrow(a[1]), most = r.narrow(a[2]);
  void* stream = read_stream(r, self, a[5]);
  return finish(r, [&] {
    return self->encode_batch(static_cast<const kvh_enc_item*>(items), n, most, kv.dt, kv.l, kv.c, &kv.v, stream);
  });
}

// decode(blob, level, n_tokens, k, v, dst_token0, page_table or None, block_tokens, status or None, stream)
PyObject* decode(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(10);
  const View kv = read_view(r, a[3], a[4], a[6] != Py_None);
  const void* blob = r.device(a[0]);
  const int level = r.narrow(a[1]), n = r.narrow(a[2]), block = r.narrow(a[7]);
  const int64_t at = r.wide(a[5]);
  const int32_t* table = r.words(a[6], 0);
  int32_t* status = r.words(a[8], 0);
  void* stream = read_stream(r, self, a[9]);
  return finish(r, [&] { return self->decode(blob, kv.dt, kv.l, n, kv.c, level, &kv.v, at, table, block, status, stream); });
}

// decode_batch(items, n_items, max_tokens_per_item, k, v, paged, block_tokens, status or None, stream)
PyObject* decode_batch(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(9);
  if (a[5] != Py_True && a[5] != Py_False) r.ok = false;
  const View kv = read_view(r, a[3], a[4], a[5] == Py_True);
  const void* items = r.device(a[0]);
  const int n = r.narrow(a[1]), most = r.narrow(a[2]), block = r.narrow(a[6]);
  int32_t* status = r.words(a[7], n);
  void* stream = read_stream(r, self, a[8]);
  return finish(r, [&] {
    return self->decode_batch(static_cast<const kvh_item*>(items), n, most, kv.dt, kv.l, kv.c, &kv.v, block, status, stream);
  });
}

// encode_kept(k, v, sink, window, level, blob, stream)
PyObject* encode_kept(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(7);
  const View kv = read_view(r, a[0], a[1], false);
  const int sink = r.narrow(a[2]), window = r.narrow(a[3]), level = r.narrow(a[4]);
  void* blob = r.device(a[5]);
  const int64_t cap = r.ok ? r.int_method(a[5], s_numel) : 0;
  void* stream = read_stream(r, self, a[6]);
  return finish(r, [&] {
    return self->encode_kept(&kv.v, kv.dt, kv.l, kv.tokens, kv.c, sink, window, level, blob, (size_t)cap, stream);
  });
}

// decode_kept(blob, level, N, sink, window, k, v, dst_token0, compact, page_table or None, block_tokens, status or None, stream)
PyObject* decode_kept(PyObject* self_, PyObject* const* a, Py_ssize_t n_args) {
  KVH_ARGS(13);
  if (a[8] != Py_True && a[8] != Py_False) r.ok = false;
  const View kv = read_view(r, a[5], a[6], a[9] != Py_None);
  const void* blob = r.device(a[0]);
  const int level = r.narrow(a[1]), n = r.narrow(a[2]), sink = r.narrow(a[3]), window = r.narrow(a[4]), block = r.narrow(a[10]);
  const int64_t at = r.wide(a[7]);
  const int32_t* table = r.words(a[9], 0);
  int32_t* status = r.words(a[11], 0);
  void* stream = read_stream(r, self, a[12]);
  return finish(r, [&] {
    return self->decode_kept(blob, kv.dt, kv.l, n, kv.c, sink, window, level, &kv.v, at, a[8] == Py_True, table, block, status, stream);
  });
}

// Calls(current_device, raw_stream, addresses of the six functions in the order of the struct)
PyObject* calls_new(PyTypeObject* type, PyObject* args, PyObject*) {
  PyObject *dev, *raw;
  unsigned long long p[6];
  if (!PyArg_ParseTuple(args, "OOKKKKKK", &dev, &raw, &p[0], &p[1], &p[2], &p[3], &p[4], &p[5])) return nullptr;
  Calls* c = reinterpret_cast<Calls*>(type->tp_alloc(type, 0));
  if (c == nullptr) return nullptr;
  c->encode = reinterpret_cast<decltype(c->encode)>((uintptr_t)p[0]);
  c->encode_batch = reinterpret_cast<decltype(c->encode_batch)>((uintptr_t)p[1]);
  c->decode = reinterpret_cast<decltype(c->decode)>((uintptr_t)p[2]);
  c->decode_batch = reinterpret_cast<decltype(c->decode_batch)>((uintptr_t)p[3]);
  c->encode_kept = reinterpret_cast<decltype(c->encode_kept)>((uintptr_t)p[4]);
  c->decode_kept = reinterpret_cast<decltype(c->decode_kept)>((uintptr_t)p[5]);
  Py_INCREF(dev);
  Py_INCREF(raw);
  c->current_device = dev;
  c->raw_stream = raw;
  return reinterpret_cast<PyObject*>(c);
}

void calls_dealloc(PyObject* o) {
  Calls* c = reinterpret_cast<Calls*>(o);
  Py_XDECREF(c->current_device);
  Py_XDECREF(c->raw_stream);
  PyTypeObject* type = Py_TYPE(o);
  type->tp_free(o);
  Py_DECREF(type);
}

#define KVH_METHOD(F) {#F, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(F)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {KVH_METHOD(encode), KVH_METHOD(encode_batch), KVH_METHOD(decode), KVH_METHOD(decode_batch),
                         KVH_METHOD(encode_kept), KVH_METHOD(decode_kept), {nullptr, nullptr, 0, nullptr}};
PyType_Slot slots[] = {{Py_tp_new, reinterpret_cast<void*>(calls_new)}, {Py_tp_dealloc, reinterpret_cast<void*>(calls_dealloc)},
                       {Py_tp_methods, methods}, {0, nullptr}};
PyType_Spec spec = {"kvh_fastcall.Calls", sizeof(Calls), 0, Py_TPFLAGS_DEFAULT, slots};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, nullptr, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) {
  PyObject* torch = PyImport_ImportModule("torch");
  if (torch == nullptr) return nullptr;
  tensor_type = PyObject_GetAttrString(torch, "Tensor");
  dtype_f16 = PyObject_GetAttrString(torch, "float16");
  dtype_bf16 = PyObject_GetAttrString(torch, "bfloat16");
  dtype_i32 = PyObject_GetAttrString(torch, "int32");
  Py_DECREF(torch);
  s_is_cuda = PyUnicode_InternFromString("is_cuda");
  s_dtype = PyUnicode_InternFromString("dtype");
  s_shape = PyUnicode_InternFromString("shape");
  s_stride = PyUnicode_InternFromString("stride");
  s_data_ptr = PyUnicode_InternFromString("data_ptr");
  s_numel = PyUnicode_InternFromString("numel");
  s_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  PyObject* m = PyModule_Create(&module);
  PyObject* type = m != nullptr ? PyType_FromSpec(&spec) : nullptr;
  if (PyErr_Occurred() || type == nullptr || PyModule_AddObject(m, "Calls", type) < 0) {
    Py_XDECREF(type);
    Py_XDECREF(m);
    return nullptr;
  }
  return m;
}
