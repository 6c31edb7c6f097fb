// Argument marshalling of the Python binding in native code: checks the tensors of a call, takes their pointers and the
// current stream, and calls the C entry point.  The same checks exist in binding.py; every function here returns None when
// one of them does not hold (or an argument is not a plain tensor or integer), and the binding then goes through its
// own checks, which raise.  A decode step on a small cache is bound by the host: 11.9 us a call through ctypes, of which
// 4.5 are spent on looking at ten tensors and converting seventeen arguments.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "adamas.h"

namespace {

PyTypeObject* g_config_type = nullptr;
PyObject* g_current_device = nullptr;   // torch's own accessors, called without arguments / with the device
PyObject* g_raw_stream = nullptr;

// The entry points of the library that the binding has loaded.
decltype(&adamas_decode_step) g_decode_step = nullptr;
decltype(&adamas_decode_step_paged) g_decode_step_paged = nullptr;
decltype(&adamas_encode_keys) g_encode_keys = nullptr;
decltype(&adamas_full_attn) g_full_attn = nullptr;

struct Config {
  Py_buffer view{};
  const adamas_config* c = nullptr;
  explicit Config(PyObject* o) {
    if (Py_TYPE(o) != g_config_type) return;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) {
      PyErr_Clear();
      return;
    }
    if (view.len == (Py_ssize_t)sizeof(adamas_config)) c = static_cast<const adamas_config*>(view.buf);
  }
  ~Config() {
    if (view.obj != nullptr) PyBuffer_Release(&view);
  }
  int64_t row_bytes() const { return c->head_dim / 8 * (c->code_bits == 0 ? 2 : c->code_bits); }
};

// The pointer of a contiguous GPU tensor of this type and shape (no shape: any); None only where it is optional.
bool tensor(PyObject* o, at::ScalarType type, std::initializer_list<int64_t> shape, void** out, bool optional = false) {
  *out = nullptr;
  if (o == Py_None) return optional;
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) return false;
  if (shape.size() != 0 && t.sizes() != at::IntArrayRef(shape)) return false;
  *out = t.data_ptr();
  return true;
}

bool integer(PyObject* o, int64_t lo, int64_t hi, int64_t* out) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  *out = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0 && *out >= lo && *out <= hi;
}
constexpr int64_t kInt32Min = INT32_MIN, kInt32Max = INT32_MAX;

// The stream: an address, or None for torch's current one.
bool stream_of(PyObject* o, void** out) {
  PyObject* got = nullptr;
  if (o == Py_None) {
    PyObject* dev = PyObject_CallNoArgs(g_current_device);
    if (dev != nullptr) {
      got = PyObject_CallOneArg(g_raw_stream, dev);
      Py_DECREF(dev);
    }
    if (got == nullptr) {
      PyErr_Clear();
      return false;
    }
    o = got;
  }
  const bool ok = PyLong_Check(o);
  if (ok) *out = PyLong_AsVoidPtr(o);
  Py_XDECREF(got);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return ok;
}

int64_t batch_of(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return -1;
  const at::Tensor& t = THPVariable_Unpack(o);
  return t.dim() == 3 ? t.size(0) : -1;
}

// Tensors that have no storage (of a transform, say) throw when they are asked for it: not a plain call.
template <class F>
PyObject* guarded(F&& fn) {
  try {
    return fn();
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// fn() without the interpreter lock, as a ctypes call runs
template <class F>
PyObject* status_of(F&& fn) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

constexpr at::ScalarType kBf16 = at::kBFloat16, kByte = at::kByte, kInt = at::kInt, kLong = at::kLong, kFloat = at::kFloat;

// What the decode steps share.
struct StepArgs {
  void *q, *k_new, *v_new, *K, *V, *codes, *seq_len, *out, *idx, *workspace, *stream;
  int64_t batch, k, max_len;
  size_t workspace_bytes;
  bool take(const Config& cfg, PyObject* q_, PyObject* K_, PyObject* V_, PyObject* codes_, PyObject* len_, PyObject* k_,
            PyObject* out_, PyObject* max_, PyObject* ws_, PyObject* k_new_, PyObject* v_new_, PyObject* idx_, PyObject* stream_) {
    if (cfg.c == nullptr || (batch = batch_of(q_)) < 0 || batch > kInt32Max) return false;
    if (!integer(k_, kInt32Min, kInt32Max, &k) || !integer(max_, INT64_MIN, INT64_MAX, &max_len)) return false;
    const int64_t hq = cfg.c->num_q_heads, hkv = cfg.c->num_kv_heads, d = cfg.c->head_dim, pool = cfg.c->pool_tokens;
    if (!tensor(q_, kBf16, {batch, hq, d}, &q) || !tensor(k_new_, kBf16, {batch, hkv, d}, &k_new, true) ||
        !tensor(v_new_, kBf16, {batch, hkv, d}, &v_new, true) || !tensor(K_, kBf16, {hkv, pool, d}, &K) ||
        !tensor(V_, kBf16, {hkv, pool, d}, &V) || !tensor(codes_, kByte, {hkv, pool, cfg.row_bytes()}, &codes) ||
        !tensor(len_, kInt, {batch}, &seq_len) || !tensor(out_, kFloat, {batch, hq, d}, &out) ||
        !tensor(idx_, kInt, {batch, hq, k}, &idx, true) || !tensor(ws_, kByte, {}, &workspace))
      return false;
    workspace_bytes = (size_t)THPVariable_Unpack(ws_).numel();
    return stream_of(stream_, &stream);
  }
};

// (cfg, q, K, V, codes, seq_start, seq_len, k, out, max_seq_len, workspace, k_new, v_new, idx_out, stream)
PyObject* decode_step(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 15) Py_RETURN_NONE;
    const Config cfg(a[0]);
    StepArgs s;
    void* start;
    if (!s.take(cfg, a[1], a[2], a[3], a[4], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14]) ||
        !tensor(a[5], kLong, {s.batch}, &start))
      Py_RETURN_NONE;
    return status_of([&] {
      return g_decode_step(cfg.c, s.q, s.k_new, s.v_new, s.K, s.V, s.codes, static_cast<const int64_t*>(start),
                           static_cast<const int32_t*>(s.seq_len), (int32_t)s.batch, (int32_t)s.k, static_cast<float*>(s.out),
                           static_cast<int32_t*>(s.idx), s.max_len, s.workspace, s.workspace_bytes, s.stream);
    });
  });
}

// (cfg, q, K, V, codes, page_table, page_tokens, seq_len, k, out, max_seq_len, workspace, k_new, v_new, idx_out, stream, stages)
PyObject* decode_step_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 17) Py_RETURN_NONE;
    const Config cfg(a[0]);
    StepArgs s;
    void* table;
    int64_t page_tokens, stages;
    if (!s.take(cfg, a[1], a[2], a[3], a[4], a[7], a[8], a[9], a[10], a[11], a[12], a[13], a[14], a[15]) ||
        !tensor(a[5], kInt, {}, &table) || !integer(a[6], kInt32Min, kInt32Max, &page_tokens) || !integer(a[16], 0, kInt32Max, &stages))
      Py_RETURN_NONE;
    const at::Tensor& t = THPVariable_Unpack(a[5]);
    if (t.dim() != 2 || t.size(0) != s.batch || t.size(1) > kInt32Max) Py_RETURN_NONE;
    const int32_t max_pages = (int32_t)t.size(1);
    return status_of([&] {
      return g_decode_step_paged(cfg.c, s.q, s.k_new, s.v_new, s.K, s.V, s.codes, static_cast<const int32_t*>(table), max_pages,
                                 (int32_t)page_tokens, static_cast<const int32_t*>(s.seq_len), (int32_t)s.batch, (int32_t)s.k,
                                 static_cast<float*>(s.out), static_cast<int32_t*>(s.idx), s.max_len, s.workspace,
                                 s.workspace_bytes, s.stream, (uint32_t)stages);
    });
  });
}

// (cfg, K, codes, row_begin, n_rows, stream)
PyObject* encode_keys(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 6) Py_RETURN_NONE;
    const Config cfg(a[0]);
    if (cfg.c == nullptr) Py_RETURN_NONE;
    const int64_t hkv = cfg.c->num_kv_heads, pool = cfg.c->pool_tokens;
    void *K, *codes, *stream;
    int64_t begin, rows;
    if (!tensor(a[1], kBf16, {hkv, pool, cfg.c->head_dim}, &K) || !tensor(a[2], kByte, {hkv, pool, cfg.row_bytes()}, &codes) ||
        !integer(a[3], INT64_MIN, INT64_MAX, &begin) || !integer(a[4], INT64_MIN, INT64_MAX, &rows) || !stream_of(a[5], &stream))
      Py_RETURN_NONE;
    return status_of([&] { return g_encode_keys(cfg.c, K, codes, begin, rows, stream); });
  });
}

// (cfg, q, K, V, seq_start, seq_len, out, max_seq_len, workspace, stream)
PyObject* full_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 10) Py_RETURN_NONE;
    const Config cfg(a[0]);
    const int64_t batch = batch_of(a[1]);
    if (cfg.c == nullptr || batch < 0 || batch > kInt32Max) Py_RETURN_NONE;
    const int64_t hq = cfg.c->num_q_heads, hkv = cfg.c->num_kv_heads, d = cfg.c->head_dim, pool = cfg.c->pool_tokens;
    void *q, *K, *V, *start, *len, *out, *ws, *stream;
    int64_t max_len;
    if (!tensor(a[1], kBf16, {batch, hq, d}, &q) || !tensor(a[2], kBf16, {hkv, pool, d}, &K) ||
        !tensor(a[3], kBf16, {hkv, pool, d}, &V) || !tensor(a[4], kLong, {batch}, &start) || !tensor(a[5], kInt, {batch}, &len) ||
        !tensor(a[6], kFloat, {batch, hq, d}, &out) || !integer(a[7], INT64_MIN, INT64_MAX, &max_len) ||
        !tensor(a[8], kByte, {}, &ws) || !stream_of(a[9], &stream))
      Py_RETURN_NONE;
    const size_t bytes = (size_t)THPVariable_Unpack(a[8]).numel();
    return status_of([&] {
      return g_full_attn(cfg.c, q, K, V, static_cast<const int64_t*>(start), static_cast<const int32_t*>(len), (int32_t)batch,
                         static_cast<float*>(out), max_len, ws, bytes, stream);
    });
  });
}

// (Config type, torch._C._cuda_getDevice, torch._C._cuda_getCurrentRawStream, addresses of the four entry points)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *type, *device, *stream;
  unsigned long long step, paged, encode, full;
  if (!PyArg_ParseTuple(args, "OOOKKKK", &type, &device, &stream, &step, &paged, &encode, &full)) return nullptr;
  if (!PyType_Check(type)) {
    PyErr_SetString(PyExc_TypeError, "the first argument must be a type");
    return nullptr;
  }
  Py_INCREF(type);
  Py_INCREF(device);
  Py_INCREF(stream);
  g_config_type = reinterpret_cast<PyTypeObject*>(type);
  g_current_device = device;
  g_raw_stream = stream;
  g_decode_step = reinterpret_cast<decltype(g_decode_step)>(step);
  g_decode_step_paged = reinterpret_cast<decltype(g_decode_step_paged)>(paged);
  g_encode_keys = reinterpret_cast<decltype(g_encode_keys)>(encode);
  g_full_attn = reinterpret_cast<decltype(g_full_attn)>(full);
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"decode_step", (PyCFunction)(void (*)(void))decode_step, METH_FASTCALL, nullptr},
    {"decode_step_paged", (PyCFunction)(void (*)(void))decode_step_paged, METH_FASTCALL, nullptr},
    {"encode_keys", (PyCFunction)(void (*)(void))encode_keys, METH_FASTCALL, nullptr},
    {"full_attn", (PyCFunction)(void (*)(void))full_attn, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr},
};

PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) {
  PyObject* m = PyModule_Create(&kModule);
  if (m != nullptr && PyModule_AddStringConstant(m, "SOURCE_ID", ADAMAS_MARSHAL_ID) != 0) Py_CLEAR(m);
  return m;
}
