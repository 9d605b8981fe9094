// Argument marshalling of the entry points that a program calls once per layer and token, as a CPython extension:
// the C structs are filled from the Python objects' attributes anew on every call and nothing is kept between calls.  What a
// library's calls need (its addresses, where the stream comes from) belongs to the functions that bind() returns for it.
// Through ctypes the structs and pointer conversions cost 3.5 us of a call's 5.5, more than the 4 us that a small layer's
// decode step takes the GPU; here 1 us.  (The launch itself, inside the C entry point, is the other 2 us.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <new>

#include "keepkv.h"

namespace {

struct Library {
  decltype(&keepkv_decode_step) decode_step;
  decltype(&keepkv_decode_step_static) decode_step_static;
  decltype(&keepkv_decode_attn) decode_attn;
  decltype(&keepkv_score) score;
  PyObject *raw_stream, *device;                     // current stream's handle of a device, current device
  PyObject* argument_error;                          // what an argument of the wrong type raises
};
const char kLibrary[] = "keepkv library";
const Library* library_of(PyObject* self) { return static_cast<const Library*>(PyCapsule_GetPointer(self, kLibrary)); }

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
bool call_uint(PyObject* obj, Name method, PyObject* error, uint64_t* out) {   // (modulo 2^64; None is 0, as ctypes takes it for an address)
  PyObject* v = PyObject_CallMethodNoArgs(obj, g_names[method]);
  if (!v) return false;
  const bool ok = v == Py_None || PyLong_Check(v);
  if (ok) *out = v == Py_None ? 0 : PyLong_AsUnsignedLongLongMask(v);
  else PyErr_Format(error, "int expected instead of %.80s instance", Py_TYPE(v)->tp_name);
  Py_DECREF(v);
  return ok && !PyErr_Occurred();
}
bool address(PyObject* tensor, PyObject* error, void** out) {         // tensor.data_ptr()
  uint64_t a = 0;
  const bool ok = call_uint(tensor, kDataPtr, error, &a);
  *out = reinterpret_cast<void*>(a);
  return ok;
}
bool address_or_null(const Library* lib, PyObject* tensor, void** out) {
  *out = nullptr;
  return tensor == Py_None || address(tensor, lib->argument_error, out);
}
bool bytes_of(const Library* lib, PyObject* tensor, size_t* out) {       // 0 for None
  uint64_t n = 0, e = 0;
  *out = 0;
  if (tensor == Py_None) return true;
  if (!call_uint(tensor, kNumel, lib->argument_error, &n) || !call_uint(tensor, kElementSize, lib->argument_error, &e)) return false;
  *out = n * e;
  return true;
}
bool float_argument(const Library* lib, PyObject* v, float* out) {
  if (to_float(v, out)) return true;
  if (PyErr_ExceptionMatches(PyExc_TypeError)) PyErr_Format(lib->argument_error, "float expected instead of %.80s instance", Py_TYPE(v)->tp_name);
  return false;
}
bool tensor_field(PyObject* obj, Name name, void** out) {
  PyObject* t = PyObject_GetAttr(obj, g_names[name]);
  const bool ok = t && address(t, PyExc_TypeError, out);
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
bool current_stream(const Library* lib, void** out) {
  PyObject* device = PyObject_CallNoArgs(lib->device);
  PyObject* s = device ? PyObject_CallOneArg(lib->raw_stream, device) : nullptr;
  if (s) *out = reinterpret_cast<void*>(PyLong_AsUnsignedLongLong(s));
  Py_XDECREF(device);
  Py_XDECREF(s);
  return s && !PyErr_Occurred();
}
bool arity(const char* name, Py_ssize_t have, Py_ssize_t want) {
  if (have == want) return true;
  PyErr_Format(PyExc_TypeError, "%s: %zd arguments, %zd expected", name, have, want);
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
PyObject* decode_step(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  const Library* lib = library_of(self);
  keepkv_layout L;
  keepkv_cache c;
  void *q, *k_t, *v_t, *out, *logits, *overflow, *ws, *stream;
  float alpha;
  size_t ws_bytes;
  if (!lib || !arity("decode_step", n, 10) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(lib, a[2], &q) ||
      !address_or_null(lib, a[3], &k_t) || !address_or_null(lib, a[4], &v_t) || !address_or_null(lib, a[5], &out) || !address_or_null(lib, a[6], &logits) ||
      !float_argument(lib, a[7], &alpha) || !address_or_null(lib, a[8], &overflow) || !address_or_null(lib, a[9], &ws) || !bytes_of(lib, a[9], &ws_bytes) ||
      !current_stream(lib, &stream))
    return nullptr;
  return status_of([&] {
    return lib->decode_step(&L, &c, q, k_t, v_t, out, static_cast<float*>(logits), alpha, static_cast<int32_t*>(overflow), ws, ws_bytes, stream);
  });
}

// (layout, cache, q, k_t, v_t, out, logits_out, alpha, overflow)
PyObject* decode_step_static(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  const Library* lib = library_of(self);
  keepkv_layout L;
  keepkv_cache c;
  void *q, *k_t, *v_t, *out, *logits, *overflow, *stream;
  float alpha;
  if (!lib || !arity("decode_step_static", n, 9) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(lib, a[2], &q) ||
      !address_or_null(lib, a[3], &k_t) || !address_or_null(lib, a[4], &v_t) || !address_or_null(lib, a[5], &out) || !address_or_null(lib, a[6], &logits) ||
      !float_argument(lib, a[7], &alpha) || !address_or_null(lib, a[8], &overflow) || !current_stream(lib, &stream))
    return nullptr;
  return status_of([&] {
    return lib->decode_step_static(&L, &c, q, k_t, v_t, out, static_cast<float*>(logits), alpha, static_cast<int32_t*>(overflow), stream);
  });
}

// (layout, cache, q, out, logits_out, lse_out, workspace)
PyObject* decode_attn(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  const Library* lib = library_of(self);
  keepkv_layout L;
  keepkv_cache c;
  void *q, *out, *logits, *lse, *ws, *stream;
  size_t ws_bytes;
  if (!lib || !arity("decode_attn", n, 7) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(lib, a[2], &q) ||
      !address_or_null(lib, a[3], &out) || !address_or_null(lib, a[4], &logits) || !address_or_null(lib, a[5], &lse) || !address_or_null(lib, a[6], &ws) ||
      !bytes_of(lib, a[6], &ws_bytes) || !current_stream(lib, &stream))
    return nullptr;
  return status_of([&] {
    return lib->decode_attn(&L, &c, q, out, static_cast<float*>(logits), static_cast<float*>(lse), ws, ws_bytes, stream);
  });
}

// (layout, cache, logits, alpha)
PyObject* score(PyObject* self, PyObject* const* a, Py_ssize_t n) {
  const Library* lib = library_of(self);
  keepkv_layout L;
  keepkv_cache c;
  void *logits, *stream;
  float alpha;
  if (!lib || !arity("score", n, 4) || !layout_of(a[0], &L) || !cache_of(a[1], &c) || !address_or_null(lib, a[2], &logits) || !float_argument(lib, a[3], &alpha) ||
      !current_stream(lib, &stream))
    return nullptr;
  return status_of([&] { return lib->score(&L, &c, static_cast<const float*>(logits), alpha, stream); });
}

PyMethodDef kCalls[] = {
    {"decode_step", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step)), METH_FASTCALL, nullptr},
    {"decode_step_static", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_step_static)), METH_FASTCALL, nullptr},
    {"decode_attn", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode_attn)), METH_FASTCALL, nullptr},
    {"score", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(score)), METH_FASTCALL, nullptr}};

void release(PyObject* capsule) {
  Library* lib = static_cast<Library*>(PyCapsule_GetPointer(capsule, kLibrary));
  Py_XDECREF(lib->raw_stream);
  Py_XDECREF(lib->device);
  Py_XDECREF(lib->argument_error);
  delete lib;
}

// (raw_stream, device, argument_error, addresses of keepkv_decode_step, keepkv_decode_step_static, keepkv_decode_attn, keepkv_score):
// these four functions for the library that the binding has loaded
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long f[4];
  PyObject *raw_stream, *device, *argument_error;
  if (!PyArg_ParseTuple(args, "OOOKKKK", &raw_stream, &device, &argument_error, &f[0], &f[1], &f[2], &f[3])) return nullptr;
  Library* lib = new (std::nothrow) Library{reinterpret_cast<decltype(&keepkv_decode_step)>(f[0]),
                                            reinterpret_cast<decltype(&keepkv_decode_step_static)>(f[1]),
                                            reinterpret_cast<decltype(&keepkv_decode_attn)>(f[2]),
                                            reinterpret_cast<decltype(&keepkv_score)>(f[3]), raw_stream, device, argument_error};
  if (!lib) return PyErr_NoMemory();
  PyObject* capsule = PyCapsule_New(lib, kLibrary, release);
  if (!capsule) {
    delete lib;
    return nullptr;
  }
  Py_INCREF(raw_stream);
  Py_INCREF(device);
  Py_INCREF(argument_error);
  PyObject* calls = PyTuple_New(4);
  for (int i = 0; calls && i < 4; ++i) {
    PyObject* call = PyCFunction_New(&kCalls[i], capsule);     // (holds the capsule)
    if (call) PyTuple_SET_ITEM(calls, i, call);
    else Py_CLEAR(calls);
  }
  Py_DECREF(capsule);
  return calls;
}

PyMethodDef kMethods[] = {{"bind", bind, METH_VARARGS, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_pycall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pycall() {
  for (int i = 0; i < kNames; ++i)
    if (!(g_names[i] = PyUnicode_InternFromString(kText[i]))) return nullptr;
  return PyModule_Create(&kModule);
}
