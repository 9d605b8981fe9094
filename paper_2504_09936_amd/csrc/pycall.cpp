// Argument marshalling of the entry points that a program calls once per layer and token, as a CPython extension:
// the C structs are filled from the Python objects' attributes anew on every call and nothing is kept between calls.
// Through ctypes the structs and pointer conversions cost 3.5 us of a call's 5.5, more than the 4 us that a small layer's
// decode step takes the GPU; here 1 us.  (The launch itself, inside the C entry point, is the other 2 us.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include "keepkv.h"

namespace {

decltype(&keepkv_decode_step) g_decode_step;
decltype(&keepkv_decode_step_static) g_decode_step_static;
decltype(&keepkv_decode_attn) g_decode_attn;
decltype(&keepkv_score) g_score;
PyObject *g_raw_stream, *g_device;                   // current stream's handle of a device, current device

enum Name { kBatch, kQHeads, kKvHeads, kHeadDim, kDtype, kScale, kK, kV, kVotes, kLogS, kBorn, kTObs, kLen, kCapacity, kLenHint,
            kPlanSlots, kPlanWaves, kDataPtr, kNumel, kElementSize, kNames };
const char* const kText[kNames] = {"batch", "n_q_heads", "n_kv_heads", "head_dim", "dtype", "scale", "k", "v", "votes", "log_s",
                                   "born", "t_obs", "len", "capacity", "len_hint", "plan_slots_per_split", "plan_wavefronts",
                                   "data_ptr", "numel", "element_size"};
PyObject* g_names[kNames];

// Each returns false with a Python exception set.
bool to_i32(PyObject* v, int32_t* out) {             // (as a ctypes field takes it: whole numbers only, modulo 2^32)
  if (!PyLong_Check(v)) {
    PyErr_Format(PyExc_TypeError, "int expected instead of %.80s instance", Py_TYPE(v)->tp_name);
    return false;
  }
  *out = (int32_t)PyLong_AsUnsignedLongMask(v);
  return !PyErr_Occurred();
}
bool int_field(PyObject* obj, Name name, int32_t* out) {
  PyObject* v = PyObject_GetAttr(obj, g_names[name]);
  const bool ok = v && to_i32(v, out);
  Py_XDECREF(v);
  return ok;
}
bool converted_int_field(PyObject* obj, Name name, int32_t* out) {   // int(obj.name)
  PyObject* v = PyObject_GetAttr(obj, g_names[name]);
  if (v && !PyLong_CheckExact(v)) {
    PyObject* i = PyNumber_Long(v);
    Py_DECREF(v);
    v = i;
  }
  const bool ok = v && to_i32(v, out);
  Py_XDECREF(v);
  return ok;
}
bool to_float(PyObject* v, float* out) {
  const double d = PyFloat_AsDouble(v);
  if (d == -1.0 && PyErr_Occurred()) return false;
  *out = (float)d;
  return true;
}
template <typename U>
bool call_uint(PyObject* obj, Name method, U* out) {
  PyObject* v = PyObject_CallMethodNoArgs(obj, g_names[method]);
  if (!v) return false;
  *out = (U)PyLong_AsUnsignedLongLong(v);
  Py_DECREF(v);
  return !PyErr_Occurred();
}
bool address(PyObject* tensor, void** out) {         // tensor.data_ptr()
  unsigned long long a = 0;
  const bool ok = call_uint(tensor, kDataPtr, &a);
  *out = reinterpret_cast<void*>(a);
  return ok;
}
bool address_or_null(PyObject* tensor, void** out) {
  *out = nullptr;
  return tensor == Py_None || address(tensor, out);
}
bool bytes_of(PyObject* tensor, size_t* out) {       // 0 for None
  size_t n = 0, e = 0;
  *out = 0;
  if (tensor == Py_None) return true;
  if (!call_uint(tensor, kNumel, &n) || !call_uint(tensor, kElementSize, &e)) return false;
  *out = n * e;
  return true;
}
bool tensor_field(PyObject* obj, Name name, void** out) {
  PyObject* t = PyObject_GetAttr(obj, g_names[name]);
  const bool ok = t && address(t, out);
  Py_XDECREF(t);
  return ok;
}
bool layout_of(PyObject* obj, keepkv_layout* L) {
  if (!int_field(obj, kBatch, &L->batch) || !int_field(obj, kQHeads, &L->n_q_heads) || !int_field(obj, kKvHeads, &L->n_kv_heads) ||
      !int_field(obj, kHeadDim, &L->head_dim) || !int_field(obj, kDtype, &L->dtype))
    return false;
  PyObject* v = PyObject_GetAttr(obj, g_names[kScale]);
  const bool ok = v && to_float(v, &L->scale);
  Py_XDECREF(v);
  return ok;
}
bool cache_of(PyObject* obj, keepkv_cache* c) {
  return tensor_field(obj, kK, &c->k) && tensor_field(obj, kV, &c->v) && tensor_field(obj, kVotes, reinterpret_cast<void**>(&c->votes)) &&
         tensor_field(obj, kLogS, reinterpret_cast<void**>(&c->log_s)) && tensor_field(obj, kBorn, reinterpret_cast<void**>(&c->born)) &&
         tensor_field(obj, kTObs, reinterpret_cast<void**>(&c->t_obs)) && tensor_field(obj, kLen, reinterpret_cast<void**>(&c->len)) &&
         int_field(obj, kCapacity, &c->capacity) && converted_int_field(obj, kLenHint, &c->len_hint) &&
         converted_int_field(obj, kPlanSlots, &c->plan_slots_per_split) && converted_int_field(obj, kPlanWaves, &c->plan_wavefronts);
}
bool current_stream(void** out) {
  PyObject* device = PyObject_CallNoArgs(g_device);
  PyObject* s = device ? PyObject_CallOneArg(g_raw_stream, device) : nullptr;
  if (s) *out = reinterpret_cast<void*>(PyLong_AsUnsignedLongLong(s));
  Py_XDECREF(device);
  Py_XDECREF(s);
  return s && !PyErr_Occurred();
}
bool arity(const char* name, Py_ssize_t have, Py_ssize_t want) {
  if (have == want && g_device) return true;
  PyErr_Format(PyExc_TypeError, "%s: %zd arguments, %zd expected (after bind)", name, have, want);
  return false;
}
template <typename F>
PyObject* status_of(F call) {                        // without the interpreter's lock, as ctypes calls
  keepkv_status st;
  Py_BEGIN_ALLOW_THREADS
  st = call();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong((long)st);
}

// (layout, cache, q, k_t, v_t, out, logits_out, alpha, overflow, workspace)
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  keepkv_layout L;
  keepkv_cache c;
  void *q, *k_t, *v_t, *out, *logits, *overflow, *ws, *stream;
  float alpha;
  size_t ws_bytes;
  if (!arity("decode_step", n, 10) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(a[2], &q) ||
      !address_or_null(a[3], &k_t) || !address_or_null(a[4], &v_t) || !address_or_null(a[5], &out) || !address_or_null(a[6], &logits) ||
      !to_float(a[7], &alpha) || !address_or_null(a[8], &overflow) || !address_or_null(a[9], &ws) || !bytes_of(a[9], &ws_bytes) ||
      !current_stream(&stream))
    return nullptr;
  return status_of([&] {
    return g_decode_step(&L, &c, q, k_t, v_t, out, static_cast<float*>(logits), alpha, static_cast<int32_t*>(overflow), ws, ws_bytes, stream);
  });
}

// (layout, cache, q, k_t, v_t, out, logits_out, alpha, overflow)
PyObject* decode_step_static(PyObject*, PyObject* const* a, Py_ssize_t n) {
  keepkv_layout L;
  keepkv_cache c;
  void *q, *k_t, *v_t, *out, *logits, *overflow, *stream;
  float alpha;
  if (!arity("decode_step_static", n, 9) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(a[2], &q) ||
      !address_or_null(a[3], &k_t) || !address_or_null(a[4], &v_t) || !address_or_null(a[5], &out) || !address_or_null(a[6], &logits) ||
      !to_float(a[7], &alpha) || !address_or_null(a[8], &overflow) || !current_stream(&stream))
    return nullptr;
  return status_of([&] {
    return g_decode_step_static(&L, &c, q, k_t, v_t, out, static_cast<float*>(logits), alpha, static_cast<int32_t*>(overflow), stream);
  });
}

// (layout, cache, q, out, logits_out, lse_out, workspace)
PyObject* decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  keepkv_layout L;
  keepkv_cache c;
  void *q, *out, *logits, *lse, *ws, *stream;
  size_t ws_bytes;
  if (!arity("decode_attn", n, 7) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(a[2], &q) ||
      !address_or_null(a[3], &out) || !address_or_null(a[4], &logits) || !address_or_null(a[5], &lse) || !address_or_null(a[6], &ws) ||
      !bytes_of(a[6], &ws_bytes) || !current_stream(&stream))
    return nullptr;
  return status_of([&] {
    return g_decode_attn(&L, &c, q, out, static_cast<float*>(logits), static_cast<float*>(lse), ws, ws_bytes, stream);
  });
}

// (layout, cache, logits, alpha)
PyObject* score(PyObject*, PyObject* const* a, Py_ssize_t n) {
  keepkv_layout L;
  keepkv_cache c;
  void *logits, *stream;
  float alpha;
  if (!arity("score", n, 4) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(a[2], &logits) || !to_float(a[3], &alpha) ||
      !current_stream(&stream))
    return nullptr;
  return status_of([&] { return g_score(&L, &c, static_cast<const float*>(logits), alpha, stream); });
}

// (raw_stream, device, addresses of keepkv_decode_step, keepkv_decode_step_static, keepkv_decode_attn, keepkv_score): once,
// at import, from the library that the binding has loaded
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[4];
  PyObject *raw_stream, *device;
  if (!PyArg_ParseTuple(args, "OOKKKK", &raw_stream, &device, &f[0], &f[1], &f[2], &f[3])) return nullptr;
  g_decode_step = reinterpret_cast<decltype(g_decode_step)>(f[0]);
  g_decode_step_static = reinterpret_cast<decltype(g_decode_step_static)>(f[1]);
  g_decode_attn = reinterpret_cast<decltype(g_decode_attn)>(f[2]);
  g_score = reinterpret_cast<decltype(g_score)>(f[3]);
  Py_INCREF(raw_stream);
  Py_INCREF(device);
  Py_XSETREF(g_raw_stream, raw_stream);
  Py_XSETREF(g_device, device);
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL, nullptr},
    {"decode_step_static", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step_static)), METH_FASTCALL, nullptr},
    {"decode_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_attn)), METH_FASTCALL, nullptr},
    {"score", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(score)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall() {
  for (int i = 0; i < kNames; ++i)
    if (!(g_names[i] = PyUnicode_InternFromString(kText[i]))) return nullptr;
  return PyModule_Create(&kModule);
}
