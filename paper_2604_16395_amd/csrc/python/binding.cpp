// Argument marshalling of the per-step calls (append, plan, attention, merge) for the Python
// package, through the CPython API: a step of small sizes is bound by what the host does between
// its launches, and building the argument structs through ctypes took 9 of the 14 us of a call.
// Every pointer, length and stream is read from the objects on each call; nothing is kept.
//
// Each function returns the library's status, or None where an argument is not of the plain form
// expected here (another type, layout or element type): the caller then takes the ctypes path,
// which words the errors.  The library's functions are handed over as addresses by setup(), so
// that this module follows the library that the package loaded.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "s2l.h"

namespace {

struct Entry {
  s2l_status (*append)(const s2l_kv_cache*, const s2l_batch*, const void*, const void*, void*);
  s2l_status (*plan)(const s2l_batch*, int32_t, int32_t, const s2l_plan_opts*, void*, size_t, s2l_plan_info*, void*);
  s2l_status (*attn[3])(const s2l_kv_cache*, const s2l_batch*, const void*, int32_t, float, void*, float*,
                        const s2l_plan_info*, void*, size_t, void*);   // attention, quantised Q, without the merge
  s2l_status (*fused)(const s2l_kv_cache*, const s2l_batch*, const void*, const void*, const void*, int32_t, float,
                      void*, float*, const s2l_plan_info*, void*, size_t, int32_t*, void*);
  s2l_status (*reduce)(const s2l_batch*, int32_t, void*, float*, const s2l_plan_info*, const void*, size_t, void*);
} lib;

PyObject *tensor_type, *cache_type, *batch_type, *opts_type, *info_type, *stream_type, *bf16, *f32, *u8, *is_initialized, *get_device, *get_stream;
PyObject *s_dtype, *s_data_ptr, *s_is_contiguous, *s_shape, *s_numel, *s_k_pages, *s_v_pages, *s_k_scale, *s_v_scale,
    *s_fp8, *s_prefix_host, *s_chunk_host, *s_tables_host, *s_prefix_lens, *s_chunk_lens, *s_cu_chunk, *s_block_tables,
    *s_cuda_stream;

// Owned reference, released at the end of the scope.
struct Ref {
  PyObject* o;
  explicit Ref(PyObject* p) : o(p) {}
  Ref(const Ref&) = delete;
  ~Ref() { Py_XDECREF(o); }
  explicit operator bool() const { return o != nullptr; }
};

bool to_ptr(PyObject* number, void** p) {
  *p = PyLong_AsVoidPtr(number);
  return !PyErr_Occurred();
}

bool data_ptr(PyObject* t, void** p) {
  const Ref v(PyObject_CallMethodNoArgs(t, s_data_ptr));
  return v && PyLong_CheckExact(v.o) && to_ptr(v.o, p);
}

// A contiguous tensor of the element type; None only where allowed (a NULL pointer).
bool tensor(PyObject* t, PyObject* dtype, void** p, bool none_ok = false) {
  *p = nullptr;
  if (t == Py_None) return none_ok;
  if ((PyObject*)Py_TYPE(t) != tensor_type) return false;
  const Ref d(PyObject_GetAttr(t, s_dtype));
  if (!d || d.o != dtype) return false;
  const Ref c(PyObject_CallMethodNoArgs(t, s_is_contiguous));
  return c && c.o == Py_True && data_ptr(t, p);
}

bool attr_data_ptr(PyObject* o, PyObject* name, void** p) {
  const Ref t(PyObject_GetAttr(o, name));
  return t && (PyObject*)Py_TYPE(t.o) == tensor_type && data_ptr(t.o, p);
}

bool numel(PyObject* t, size_t* n) {
  const Ref v(PyObject_CallMethodNoArgs(t, s_numel));
  if (!v) return false;
  *n = PyLong_AsSize_t(v.o);
  return !PyErr_Occurred();
}

// A contiguous int32 buffer held by an attribute (a numpy array).
struct HostArray {
  Py_buffer b{};
  bool held = false;
  ~HostArray() {
    if (held) PyBuffer_Release(&b);
  }
  bool take(PyObject* o, PyObject* name, int ndim) {
    const Ref a(PyObject_GetAttr(o, name));
    if (!a || PyObject_GetBuffer(a.o, &b, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) return false;
    held = true;
    return b.ndim == ndim && b.itemsize == 4 && b.format && b.format[0] == 'i' && b.format[1] == 0;
  }
};

struct BatchArg {
  s2l_batch c{};
  HostArray prefix, chunk;
  bool take(PyObject* o) {
    if ((PyObject*)Py_TYPE(o) != batch_type) return false;
    HostArray tables;
    void* p[4];
    if (!prefix.take(o, s_prefix_host, 1) || !chunk.take(o, s_chunk_host, 1) || !tables.take(o, s_tables_host, 2) ||
        chunk.b.shape[0] != prefix.b.shape[0] || tables.b.shape[1] > INT32_MAX ||
        !attr_data_ptr(o, s_prefix_lens, &p[0]) || !attr_data_ptr(o, s_chunk_lens, &p[1]) ||
        !attr_data_ptr(o, s_cu_chunk, &p[2]) || !attr_data_ptr(o, s_block_tables, &p[3]))
      return false;
    c.num_reqs = (int32_t)prefix.b.shape[0];
    c.max_pages_per_req = (int32_t)tables.b.shape[1];
    c.prefix_lens = static_cast<const int32_t*>(p[0]);
    c.chunk_lens = static_cast<const int32_t*>(p[1]);
    c.cu_chunk = static_cast<const int32_t*>(p[2]);
    c.block_tables = static_cast<const int32_t*>(p[3]);
    c.prefix_lens_host = static_cast<const int32_t*>(prefix.b.buf);
    c.chunk_lens_host = static_cast<const int32_t*>(chunk.b.buf);
    return true;
  }
};

bool cache_arg(PyObject* o, s2l_kv_cache* c) {
  if ((PyObject*)Py_TYPE(o) != cache_type) return false;
  *c = s2l_kv_cache{};
  const Ref k(PyObject_GetAttr(o, s_k_pages)), fp8(PyObject_GetAttr(o, s_fp8));
  if (!k || !fp8 || (PyObject*)Py_TYPE(k.o) != tensor_type || (fp8.o != Py_True && fp8.o != Py_False)) return false;
  const Ref shape(PyObject_GetAttr(k.o, s_shape));
  if (!shape || !PyTuple_Check(shape.o) || PyTuple_GET_SIZE(shape.o) != 4) return false;
  int32_t n[4];
  for (int i = 0; i < 4; ++i) {
    const long long x = PyLong_AsLongLong(PyTuple_GET_ITEM(shape.o, i));
    if (PyErr_Occurred() || x < 0 || x > INT32_MAX) return false;
    n[i] = (int32_t)x;
  }
  void *ks = nullptr, *vs = nullptr;
  if (!data_ptr(k.o, &c->k_pages) || !attr_data_ptr(o, s_v_pages, &c->v_pages)) return false;
  if (fp8.o == Py_True && (!attr_data_ptr(o, s_k_scale, &ks) || !attr_data_ptr(o, s_v_scale, &vs))) return false;
  c->k_scale = static_cast<const float*>(ks);
  c->v_scale = static_cast<const float*>(vs);
  c->num_pages = n[0];
  c->num_kv_heads = n[1];
  c->page_size = n[2];
  c->head_dim = n[3];
  c->dtype = fp8.o == Py_True ? S2L_KV_FP8_E4M3 : S2L_KV_BF16;
  return true;
}

// None: the current stream of the current device; a number; or a torch.cuda.Stream.
bool stream_arg(PyObject* s, void** p) {
  if (s == Py_None) {
    const Ref ready(PyObject_CallNoArgs(is_initialized));
    if (!ready || ready.o != Py_True) return false;
    const Ref dev(PyObject_CallNoArgs(get_device));
    if (!dev) return false;
    const Ref raw(PyObject_CallOneArg(get_stream, dev.o));
    return raw && to_ptr(raw.o, p);
  }
  if (PyLong_CheckExact(s)) return to_ptr(s, p);
  if (PyObject_IsInstance(s, stream_type) != 1) return false;
  const Ref raw(PyObject_GetAttr(s, s_cuda_stream));
  return raw && PyLong_CheckExact(raw.o) && to_ptr(raw.o, p);
}

// A ctypes structure of exactly this type; None only where allowed.
template <typename T>
struct StructArg {
  Py_buffer b{};
  bool held = false;
  T* p = nullptr;
  ~StructArg() {
    if (held) PyBuffer_Release(&b);
  }
  bool take(PyObject* o, PyObject* type, bool none_ok = false) {
    if (o == Py_None) return none_ok;
    if ((PyObject*)Py_TYPE(o) != type || PyObject_GetBuffer(o, &b, PyBUF_WRITABLE) != 0) return false;
    held = true;
    p = static_cast<T*>(b.buf);
    return b.len == (Py_ssize_t)sizeof(T);
  }
};

bool int_arg(PyObject* o, int32_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  const long x = PyLong_AsLong(o);
  if (PyErr_Occurred() || x < INT32_MIN || x > INT32_MAX) return false;
  *v = (int32_t)x;
  return true;
}

PyObject* general() {   // not the plain form: whatever was raised on the way does not count
  PyErr_Clear();
  Py_RETURN_NONE;
}

template <typename F>
PyObject* call(F f) {
  s2l_status st;
  Py_BEGIN_ALLOW_THREADS st = f();
  Py_END_ALLOW_THREADS return PyLong_FromLong(st);
}

// (cache, batch, k_new, v_new, stream)
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  s2l_kv_cache cache;
  BatchArg batch;
  void *k, *v, *stream;
  if (n != 5 || !tensor(a[2], bf16, &k) || !tensor(a[3], bf16, &v) || !cache_arg(a[0], &cache) || !batch.take(a[1]) ||
      !stream_arg(a[4], &stream))
    return general();
  return call([&] { return lib.append(&cache, &batch.c, k, v, stream); });
}

// (batch, hq, hkv, opts, workspace, info, stream)
PyObject* plan(PyObject*, PyObject* const* a, Py_ssize_t n) {
  BatchArg batch;
  StructArg<s2l_plan_opts> opts;
  StructArg<s2l_plan_info> info;
  int32_t hq, hkv;
  void *ws, *stream;
  size_t bytes;
  if (n != 7 || !batch.take(a[0]) || !int_arg(a[1], &hq) || !int_arg(a[2], &hkv) || !opts.take(a[3], opts_type, true) ||
      !tensor(a[4], u8, &ws) || !numel(a[4], &bytes) || !info.take(a[5], info_type) || !stream_arg(a[6], &stream))
    return general();
  return call([&] { return lib.plan(&batch.c, hq, hkv, opts.p, ws, bytes, info.p, stream); });
}

struct AttnArgs {
  s2l_kv_cache cache;
  BatchArg batch;
  StructArg<s2l_plan_info> plan;
  void *q, *out, *lse, *ws, *stream;
  int32_t hq;
  size_t bytes;
  float scale;
  // (cache, batch, q, hq, scale, out, lse, plan, workspace, stream)
  bool take(PyObject* const* a) {
    if (!tensor(a[2], bf16, &q) || !tensor(a[5], bf16, &out) || !tensor(a[6], f32, &lse, true) ||
        !tensor(a[8], u8, &ws) || !numel(a[8], &bytes) || !cache_arg(a[0], &cache) || !batch.take(a[1]) ||
        !int_arg(a[3], &hq) || !PyFloat_CheckExact(a[4]) || !plan.take(a[7], info_type) || !stream_arg(a[9], &stream))
      return false;
    scale = (float)PyFloat_AS_DOUBLE(a[4]);
    return true;
  }
};

// (which, cache, batch, q, hq, scale, out, lse, plan, workspace, stream)
PyObject* attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  AttnArgs x;
  int32_t which;
  if (n != 11 || !int_arg(a[0], &which) || which < 0 || which > 2 || !x.take(a + 1)) return general();
  return call([&] {
    return lib.attn[which](&x.cache, &x.batch.c, x.q, x.hq, x.scale, x.out, static_cast<float*>(x.lse), x.plan.p, x.ws,
                           x.bytes, x.stream);
  });
}

// (cache, batch, q, hq, scale, out, lse, plan, workspace, stream, k_new, v_new): (status, fused)
PyObject* fused(PyObject*, PyObject* const* a, Py_ssize_t n) {
  AttnArgs x;
  void *k, *v;
  if (n != 12 || !tensor(a[10], bf16, &k) || !tensor(a[11], bf16, &v) || !x.take(a)) return general();
  int32_t used = 0;
  s2l_status st;
  Py_BEGIN_ALLOW_THREADS st = lib.fused(&x.cache, &x.batch.c, k, v, x.q, x.hq, x.scale, x.out,
                                        static_cast<float*>(x.lse), x.plan.p, x.ws, x.bytes, &used, x.stream);
  Py_END_ALLOW_THREADS return Py_BuildValue("(iO)", (int)st, used ? Py_True : Py_False);
}

// (batch, hq, out, lse, plan, workspace, stream)
PyObject* reduce(PyObject*, PyObject* const* a, Py_ssize_t n) {
  BatchArg batch;
  StructArg<s2l_plan_info> info;
  int32_t hq;
  void *out, *lse, *ws, *stream;
  size_t bytes;
  if (n != 7 || !tensor(a[2], bf16, &out) || !tensor(a[3], f32, &lse, true) || !tensor(a[5], u8, &ws) ||
      !numel(a[5], &bytes) || !batch.take(a[0]) || !int_arg(a[1], &hq) || !info.take(a[4], info_type) || !stream_arg(a[6], &stream))
    return general();
  return call([&] { return lib.reduce(&batch.c, hq, out, static_cast<float*>(lse), info.p, ws, bytes, stream); });
}

// (types and dtypes and torch functions as a tuple, entry point addresses as a tuple)
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
  void* f[7];
  PyObject** o[] = {&tensor_type, &cache_type, &batch_type, &opts_type, &info_type, &stream_type,
                    &bf16, &f32, &u8, &is_initialized, &get_device, &get_stream};
  if (n != 2 || !PyTuple_Check(a[0]) || PyTuple_GET_SIZE(a[0]) != 12 || !PyTuple_Check(a[1]) || PyTuple_GET_SIZE(a[1]) != 7) {
    PyErr_SetString(PyExc_TypeError, "setup(objects, addresses)");
    return nullptr;
  }
  for (int i = 0; i < 7; ++i)
    if (!to_ptr(PyTuple_GET_ITEM(a[1], i), &f[i])) return nullptr;
  for (int i = 0; i < 12; ++i) {
    Py_INCREF(PyTuple_GET_ITEM(a[0], i));
    Py_XSETREF(*o[i], PyTuple_GET_ITEM(a[0], i));
  }
  lib.append = reinterpret_cast<decltype(lib.append)>(f[0]);
  lib.plan = reinterpret_cast<decltype(lib.plan)>(f[1]);
  for (int i = 0; i < 3; ++i) lib.attn[i] = reinterpret_cast<decltype(lib.attn[0])>(f[2 + i]);
  lib.fused = reinterpret_cast<decltype(lib.fused)>(f[5]);
  lib.reduce = reinterpret_cast<decltype(lib.reduce)>(f[6]);
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(setup), FAST(append), FAST(plan), FAST(attn), FAST(fused), FAST(reduce), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", "Argument marshalling of the per-step calls.", -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  const struct {
    PyObject** o;
    const char* s;
  } names[] = {{&s_dtype, "dtype"}, {&s_data_ptr, "data_ptr"}, {&s_is_contiguous, "is_contiguous"}, {&s_shape, "shape"},
               {&s_numel, "numel"}, {&s_k_pages, "k_pages"}, {&s_v_pages, "v_pages"}, {&s_k_scale, "k_scale"},
               {&s_v_scale, "v_scale"}, {&s_fp8, "fp8"}, {&s_prefix_host, "prefix_host"}, {&s_chunk_host, "chunk_host"},
               {&s_tables_host, "tables_host"}, {&s_prefix_lens, "prefix_lens"}, {&s_chunk_lens, "chunk_lens"},
               {&s_cu_chunk, "cu_chunk"}, {&s_block_tables, "block_tables"}, {&s_cuda_stream, "cuda_stream"}};
  for (const auto& n : names)
    if (!(*n.o = PyUnicode_InternFromString(n.s))) return nullptr;
  return PyModule_Create(&module);
}
