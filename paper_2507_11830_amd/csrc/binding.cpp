// Argument marshalling of the Python entry points (CPython C API): tensors to device pointers, shapes to counts, the
// current stream to its handle, then the C-ABI call with the interpreter lock released.  Same conversions as ctypes makes.
//
// Why native.  A call of a small step is shorter on the GPU than its marshalling was through ctypes (host time per call, one
// sequence of 137 keys: 8.2 us against 4.7 us of kernel): seven data_ptr calls, two shapes, a stream object and the
// conversion of 15 arguments cost 5 us, where the launch itself costs 2 to 3.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <pthread.h>
#include <stdint.h>

#include "shiftattn.h"

namespace {

struct Entry {
  const char *name;
  void *fn;
};
enum { kAppend, kPrefill, kChunkStep, kDecode, kDecodeStatic, kDecodeStep, kEntries };
Entry entries[kEntries] = {{"sp_kv_append", nullptr},   {"sp_attn_prefill", nullptr},       {"sp_chunk_step", nullptr},
                           {"sp_attn_decode", nullptr}, {"sp_attn_decode_static", nullptr}, {"sp_decode_step", nullptr}};
PyObject *s_data_ptr, *s_shape, *s_numel, *s_element_size, *s_cuda_stream, *s_desc, *s_value, *s_as_parameter;
PyObject *argument_error, *c_int32, *desc_type;    // ctypes.ArgumentError, ctypes.c_int32, sp_cache_desc
PyObject *get_device, *get_stream, *first_stream;  // torch's raw accessors; the public one, for the first call of the process
bool stream_used = false;  // the public accessor has been called in this process

// Every helper returns false with a Python exception set.
bool pointer(PyObject *t, void **p) {
  *p = nullptr;
  if (t == Py_None) return true;
  PyObject *v = PyObject_CallMethodNoArgs(t, s_data_ptr);
  if (!v) return false;
  *p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !(*p == nullptr && PyErr_Occurred());
}

// What ctypes takes for a c_int32: one itself, an integer (out-of-range values keep their low bits), or an object that names either
// of them in _as_parameter_.
bool int32(PyObject *o, int32_t *out) {
  PyObject *v = PyFloat_Check(o) ? nullptr : PyNumber_Index(o);
  if (!v) {
    PyErr_Clear();
    const int own = PyObject_IsInstance(o, c_int32);
    PyObject *inner = own < 0 ? nullptr : PyObject_GetAttr(o, own ? s_value : s_as_parameter);
    if (!inner) {
      PyErr_Clear();
      PyErr_SetString(argument_error, "wrong type");
      return false;
    }
    const bool deep = Py_EnterRecursiveCall(" while converting an argument") != 0;
    const bool ok = !deep && int32(inner, out);
    if (!deep) Py_LeaveRecursiveCall();
    Py_DECREF(inner);
    return ok;
  }
  *out = (int32_t)PyLong_AsUnsignedLongMask(v);
  Py_DECREF(v);
  return true;
}

bool dims(PyObject *t, int32_t *out, Py_ssize_t n, bool exactly) {  // the first n sizes
  PyObject *shape = PyObject_GetAttr(t, s_shape);
  if (!shape) return false;
  PyObject *fast = PySequence_Fast(shape, "shape is not a sequence");
  Py_DECREF(shape);
  if (!fast) return false;
  const Py_ssize_t have = PySequence_Fast_GET_SIZE(fast);
  bool ok = have >= n && !(exactly && have > n);
  if (!ok) {
    if (exactly) PyErr_Format(PyExc_ValueError, "expected %zd sizes, got %zd", n, have);
    else PyErr_SetString(PyExc_IndexError, "tuple index out of range");
  }
  for (Py_ssize_t i = 0; ok && i < n; ++i) ok = int32(PySequence_Fast_GET_ITEM(fast, i), out + i);
  Py_DECREF(fast);
  return ok;
}

bool bytes_of(PyObject *t, size_t *out) {
  *out = 0;
  if (t == Py_None) return true;
  PyObject *n = PyObject_CallMethodNoArgs(t, s_numel), *e = n ? PyObject_CallMethodNoArgs(t, s_element_size) : nullptr;
  PyObject *b = e ? PyNumber_Multiply(n, e) : nullptr;
  if (b) *out = PyLong_AsSize_t(b);
  Py_XDECREF(n);
  Py_XDECREF(e);
  Py_XDECREF(b);
  return b && !(*out == (size_t)-1 && PyErr_Occurred());
}

bool stream_of(PyObject *s, void **out) {
  PyObject *v = nullptr;
  if (s == Py_None && stream_used) {
    PyObject *dev = PyObject_CallNoArgs(get_device);
    if (!dev) return false;
    v = PyObject_CallOneArg(get_stream, dev);
    Py_DECREF(dev);
  } else {
    PyObject *own = nullptr;
    if (s == Py_None) {  // the public accessor initialises torch's device state, or says why it cannot
      own = s = PyObject_CallNoArgs(first_stream);
      if (!s) return false;
      stream_used = true;
    }
    v = PyObject_GetAttr(s, s_cuda_stream);
    if (!v && PyErr_ExceptionMatches(PyExc_AttributeError)) {
      PyErr_Clear();
      v = PyNumber_Long(s);
    }
    Py_XDECREF(own);
  }
  if (!v) return false;
  *out = v == Py_None ? nullptr : PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  return !(*out == nullptr && PyErr_Occurred());
}

bool scale_of(PyObject *o, float *out) {
  PyObject *v = PyNumber_Float(o);
  if (!v) return false;
  *out = (float)PyFloat_AS_DOUBLE(v);
  Py_DECREF(v);
  return true;
}

struct Desc {  // cache.desc, a ctypes structure: its memory
  Py_buffer view;
  bool held = false;
  bool take(PyObject *cache) {
    PyObject *d = PyObject_GetAttr(cache, s_desc);
    if (!d) return false;
    const int is = PyObject_IsInstance(d, desc_type);
    if (is > 0) held = PyObject_GetBuffer(d, &view, PyBUF_SIMPLE) == 0;
    else if (is == 0) PyErr_SetString(argument_error, "cache.desc is not a cache descriptor");
    Py_DECREF(d);
    return held;
  }
  const sp_cache_desc *get() const { return (const sp_cache_desc *)view.buf; }
  ~Desc() {
    if (held) PyBuffer_Release(&view);
  }
};

bool count(const char *name, Py_ssize_t have, Py_ssize_t want) {
  if (have == want && entries[0].fn) return true;
  PyErr_Format(PyExc_TypeError, entries[0].fn ? "%s: %zd arguments, not %zd" : "%s: the library is not bound", name, want, have);
  return false;
}

template <typename Call>
PyObject *finish(Call call) {  // the status
  int status;
  Py_BEGIN_ALLOW_THREADS;
  status = call();
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(status);
}

// (cache, k_new, v_new, cu_seqlens_new, ctx_lens, block_table, stream)
PyObject *kv_append(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[5], *stream;
  int32_t table[2], total;
  if (!count("kv_append", n, 7) || !dims(a[5], table, 2, true) || !dims(a[1], &total, 1, false) || !desc.take(a[0])) return nullptr;
  for (int i = 0; i < 5; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!stream_of(a[6], &stream)) return nullptr;
  return finish([&] {
    return ((decltype(&sp_kv_append))entries[kAppend].fn)(desc.get(), p[0], p[1], (const int32_t *)p[2], (const int32_t *)p[3],
                                                          (const int32_t *)p[4], table[0], table[1], total, stream);
  });
}

// (cache, q, out, cu_seqlens_q, ctx_lens, block_table, max_q_len, max_kv_len, scale, causal, workspace, stream)
PyObject *attn_prefill(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[5], *ws, *stream;
  int32_t table[2], q[2], max_q, max_kv, causal;
  float scale;
  size_t ws_bytes;
  if (!count("attn_prefill", n, 12) || !dims(a[5], table, 2, true) || !dims(a[1], q, 2, false) || !bytes_of(a[10], &ws_bytes) || !desc.take(a[0]))
    return nullptr;
  for (int i = 0; i < 5; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!scale_of(a[8], &scale) || !pointer(a[10], &ws) || !stream_of(a[11], &stream) || !int32(a[6], &max_q) || !int32(a[7], &max_kv) ||
      !int32(a[9], &causal))
    return nullptr;
  return finish([&] {
    return ((decltype(&sp_attn_prefill))entries[kPrefill].fn)(desc.get(), p[0], p[1], (const int32_t *)p[2], (const int32_t *)p[3],
                                                              (const int32_t *)p[4], table[0], table[1], q[0], max_q, max_kv, q[1], scale, causal,
                                                              ws, ws_bytes, stream);
  });
}

// (cache, k_new, v_new, q, out, cu_seqlens_q, ctx_lens, block_table, max_q_len, max_kv_len, scale, workspace, stream)
PyObject *chunk_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[7], *ws, *stream;
  int32_t table[2], q[2], max_q, max_kv;
  float scale;
  size_t ws_bytes;
  if (!count("chunk_step", n, 13) || !dims(a[7], table, 2, true) || !dims(a[3], q, 2, false) || !bytes_of(a[11], &ws_bytes) || !desc.take(a[0]))
    return nullptr;
  for (int i = 0; i < 7; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!scale_of(a[10], &scale) || !pointer(a[11], &ws) || !stream_of(a[12], &stream) || !int32(a[8], &max_q) || !int32(a[9], &max_kv)) return nullptr;
  return finish([&] {
    return ((decltype(&sp_chunk_step))entries[kChunkStep].fn)(desc.get(), p[0], p[1], p[2], p[3], (const int32_t *)p[4], (const int32_t *)p[5],
                                                              (const int32_t *)p[6], table[0], table[1], q[0], max_q, max_kv, q[1], scale, ws,
                                                              ws_bytes, stream);
  });
}

// (cache, q, out, seq_lens, block_table, max_seq_len, scale, workspace, stream)
PyObject *attn_decode(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[4], *ws, *stream;
  int32_t table[2], q[2], max_len;
  float scale;
  size_t ws_bytes;
  if (!count("attn_decode", n, 9) || !dims(a[4], table, 2, true) || !dims(a[1], q, 2, false) || !bytes_of(a[7], &ws_bytes) || !desc.take(a[0]))
    return nullptr;
  for (int i = 0; i < 4; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!scale_of(a[6], &scale) || !pointer(a[7], &ws) || !stream_of(a[8], &stream) || !int32(a[5], &max_len)) return nullptr;
  return finish([&] {
    return ((decltype(&sp_attn_decode))entries[kDecode].fn)(desc.get(), p[0], p[1], (const int32_t *)p[2], (const int32_t *)p[3], table[0], table[1],
                                                            max_len, q[1], scale, ws, ws_bytes, stream);
  });
}

// (cache, q, out, seq_lens, block_table, max_seq_len, scale, stream)
PyObject *attn_decode_static(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[4], *stream;
  int32_t table[2], q[2], max_len;
  float scale;
  if (!count("attn_decode_static", n, 8) || !dims(a[4], table, 2, true) || !dims(a[1], q, 2, false) || !desc.take(a[0])) return nullptr;
  for (int i = 0; i < 4; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!scale_of(a[6], &scale) || !stream_of(a[7], &stream) || !int32(a[5], &max_len)) return nullptr;
  return finish([&] {
    return ((decltype(&sp_attn_decode_static))entries[kDecodeStatic].fn)(desc.get(), p[0], p[1], (const int32_t *)p[2], (const int32_t *)p[3],
                                                                         table[0], table[1], max_len, q[1], scale, stream);
  });
}

// (cache, k_new, v_new, q, out, seq_lens, block_table, max_seq_len, scale, workspace, stream)
PyObject *decode_step(PyObject *, PyObject *const *a, Py_ssize_t n) {
  Desc desc;
  void *p[6], *ws, *stream;
  int32_t table[2], q[2], max_len;
  float scale;
  size_t ws_bytes;
  if (!count("decode_step", n, 11) || !dims(a[6], table, 2, true) || !dims(a[3], q, 2, false) || !bytes_of(a[9], &ws_bytes) || !desc.take(a[0]))
    return nullptr;
  for (int i = 0; i < 6; ++i)
    if (!pointer(a[1 + i], p + i)) return nullptr;
  if (!scale_of(a[8], &scale) || !pointer(a[9], &ws) || !stream_of(a[10], &stream) || !int32(a[7], &max_len)) return nullptr;
  return finish([&] {
    return ((decltype(&sp_decode_step))entries[kDecodeStep].fn)(desc.get(), p[0], p[1], p[2], p[3], (const int32_t *)p[4], (const int32_t *)p[5],
                                                                table[0], table[1], max_len, q[1], scale, ws, ws_bytes, stream);
  });
}

// bind(addresses, ArgumentError, c_int32, sp_cache_desc, get_device, get_stream, first_stream): addresses maps the C-ABI names to the
// loaded library's functions
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *table, *values[6];
  if (!PyArg_ParseTuple(args, "O!OOOOOO", &PyDict_Type, &table, values, values + 1, values + 2, values + 3, values + 4, values + 5)) return nullptr;
  void *fn[kEntries];
  for (int i = 0; i < kEntries; ++i) {
    PyObject *v = PyDict_GetItemString(table, entries[i].name);
    if (!v) return PyErr_Format(PyExc_KeyError, "%s", entries[i].name);
    fn[i] = PyLong_AsVoidPtr(v);
    if (!fn[i]) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_ValueError, "%s is NULL", entries[i].name);
  }
  PyObject **slots[6] = {&argument_error, &c_int32, &desc_type, &get_device, &get_stream, &first_stream};
  for (int i = 0; i < 6; ++i) {
    Py_INCREF(values[i]);
    Py_XSETREF(*slots[i], values[i]);
  }
  for (int i = 0; i < kEntries; ++i) entries[i].fn = fn[i];
  Py_RETURN_NONE;
}

#define FAST(f) {#f, (PyCFunction)(void (*)(void))f, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"bind", bind, METH_VARARGS, nullptr}, FAST(kv_append), FAST(attn_prefill), FAST(chunk_step), FAST(attn_decode),
                         FAST(attn_decode_static), FAST(decode_step), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) {
  struct {
    PyObject **slot;
    const char *text;
  } names[] = {{&s_data_ptr, "data_ptr"},       {&s_shape, "shape"}, {&s_numel, "numel"}, {&s_element_size, "element_size"},
               {&s_cuda_stream, "cuda_stream"}, {&s_desc, "desc"},   {&s_value, "value"},   {&s_as_parameter, "_as_parameter_"}};
  // In a forked child torch's device state is unusable: the public accessor says so, the raw ones go on.
  static bool registered = false;
  if (!registered && pthread_atfork(nullptr, nullptr, [] { stream_used = false; }) != 0) return PyErr_NoMemory();
  registered = true;
  for (auto &x : names)
    if (!(*x.slot = PyUnicode_InternFromString(x.text))) return nullptr;
  return PyModule_Create(&module);
}
