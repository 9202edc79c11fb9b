// Argument marshalling of the Python binding in native code: tensors to apbv_tensor, the checks of the caller's buffers, the
// current stream, the call.  For the smallest problems the interpreter's time is the call's (one launch takes 2.9 us to
// enqueue; a call from Python took 3.4 us more for a merge, 7 to 8 us more for an attention).  Enqueueing, before / now
// (us): merge 6.9 / 3.4, attention 10.5 / 4.8, query attention (two launches) 16.0 / 8.1, compression (three) 15.7 / 8.3.
//
// Every function returns the call's status, or None where a call is not the plain case -- an output left to the binding to
// allocate, an argument of another type, a tensor subclass, any check that fails: the binding then goes the general way,
// which accepts or refuses it with its own message.  Nothing is kept from one call to the next.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <vector>
#include "apbv.h"

namespace {

PyObject* g_is_initialized = nullptr;      // torch.cuda.is_initialized, torch._C._cuda_getDevice, _cuda_getCurrentRawStream
PyObject* g_current_device = nullptr;
PyObject* g_raw_stream = nullptr;

PyObject* not_taken() { Py_RETURN_NONE; }

// An ordinary dense-memory tensor, or nullptr: no subclass, no wrapper of a function transform.
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || t.layout() != at::kStrided || !t.has_storage()) return nullptr;
  const auto keys = t.key_set();
  if (keys.has_any(c10::functorch_transforms_ks) || keys.has(c10::DispatchKey::Python) || keys.has(c10::DispatchKey::Functionalize) ||
      t.unsafeGetTensorImpl()->has_symbolic_sizes_strides())
    return nullptr;
  return &t;
}

// [tokens, heads, d] or [batch, tokens, heads, d] bfloat16 -> apbv_tensor and batch; false: not the plain case.
struct Tensor {
  apbv_tensor view;
  int64_t batch, tokens, heads, d;
  c10::Device device = at::kCPU;
};
bool view_of(PyObject* o, Tensor& out, int dims = 0) {
  const at::Tensor* t = plain(o);
  if (t == nullptr || t->scalar_type() != at::kBFloat16 || (dims != 0 && t->dim() != dims)) return false;
  const auto n = t->sizes(), s = t->strides();
  const int64_t dim = t->dim();
  if (dim != 3 && dim != 4) return false;
  out.batch = dim == 4 ? n[0] : 1;
  out.tokens = n[dim - 3];
  out.heads = n[dim - 2];
  out.d = n[dim - 1];
  if (out.tokens > 0 && s[dim - 1] != 1) return false;
  out.view.ptr = out.tokens > 0 ? t->data_ptr() : nullptr;
  out.view.tokens = out.tokens;
  out.view.stride_token = s[dim - 3];
  out.view.stride_head = s[dim - 2];
  out.view.stride_batch = dim == 4 ? s[0] : out.tokens * s[0];
  out.device = t->device();
  return true;
}

// A buffer the library writes: dense, of the type, on the device, holding at least `need` elements.  None gives a null
// pointer where that is allowed.
bool buffer(PyObject* o, at::ScalarType type, int64_t need, c10::Device device, bool optional, void*& ptr, int64_t* numel = nullptr) {
  ptr = nullptr;
  if (o == Py_None) return optional;
  const at::Tensor* t = plain(o);
  if (t == nullptr || t->scalar_type() != type || !t->is_cuda() || t->device() != device || !t->is_contiguous() || t->numel() < need) return false;
  ptr = t->data_ptr();
  if (numel != nullptr) *numel = t->numel();
  return true;
}

bool number(PyObject* o, float& x) {
  if (!PyFloat_CheckExact(o) && !PyLong_CheckExact(o)) return false;
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  x = (float)v;
  return true;
}
bool whole(PyObject* o, int64_t& x) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  x = PyLong_AsLongLongAndOverflow(o, &overflow);
  return overflow == 0;
}

// The current device's current stream; false if CUDA is not initialised in this process, or with what was raised (by a signal's
// handler, say: these functions run Python code).
bool current_stream(void*& stream) {
  PyObject* ok = PyObject_CallNoArgs(g_is_initialized);
  const bool ready = ok == Py_True;
  Py_XDECREF(ok);
  if (!ready) return false;
  PyObject* dev = PyObject_CallNoArgs(g_current_device);
  if (dev == nullptr) return false;
  PyObject* raw = PyObject_CallOneArg(g_raw_stream, dev);
  Py_DECREF(dev);
  if (raw == nullptr) return false;
  stream = PyLong_AsVoidPtr(raw);
  Py_DECREF(raw);
  return PyErr_Occurred() == nullptr;
}

int to_int(int64_t x) { return x > 0x7fffffff ? 0x7fffffff : (int)x; }      // sizes the library refuses either way

// Runs f (false: not the plain case), with no C++ exception leaving.
template <typename F>
PyObject* guarded(F&& f) {
  if (g_raw_stream == nullptr || at::impl::torch_function_mode_enabled()) return not_taken();
  int status = 0;
  bool taken = false;
  try {
    taken = f(status);
  } catch (...) {
    taken = false;
  }
  if (taken) return PyLong_FromLong(status);
  return PyErr_Occurred() ? nullptr : not_taken();
}

// merge_lse(parts_out, parts_lse, out, lse_out)
PyObject* merge_lse(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 4) return not_taken();
  return guarded([&](int& status) {
    const at::Tensor *po = plain(a[0]), *pl = plain(a[1]);
    if (po == nullptr || pl == nullptr || po->scalar_type() != at::kBFloat16 || pl->scalar_type() != at::kFloat || po->dim() != 4 || pl->dim() != 3) return false;
    const int64_t parts = po->size(0), rows = po->size(1), hq = po->size(2), d = po->size(3);
    if (parts < 1 || pl->size(0) != parts || pl->size(1) != hq || pl->size(2) != rows || !po->is_contiguous() || !pl->is_contiguous()) return false;
    void *out, *lse, *stream;
    if (a[2] == Py_None || !buffer(a[2], at::kBFloat16, rows * hq * d, po->device(), false, out) ||
        !buffer(a[3], at::kFloat, hq * rows, po->device(), true, lse) || !current_stream(stream))
      return false;
    const void *po_ptr = po->data_ptr(), *pl_ptr = pl->data_ptr();
    const int64_t so = po->stride(0), sl = pl->stride(0);
    Py_BEGIN_ALLOW_THREADS
    status = apbv_merge_lse(to_int(parts), rows, to_int(hq), to_int(d), po_ptr, so, static_cast<const float*>(pl_ptr), sl, out, static_cast<float*>(lse), stream);
    Py_END_ALLOW_THREADS
    return true;
  });
}

// The seven tensors of an attention call; all of one batch.
bool attention_views(PyObject* const* a, Tensor (&t)[7], int dims = 0) {
  for (int i = 0; i < 7; ++i)
    if (!view_of(a[i], t[i], dims) || t[i].batch != t[0].batch) return false;
  return true;
}

// host_attention(seven tensors, scale, out, lse_out)
PyObject* host_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 10) return not_taken();
  return guarded([&](int& status) {
    Tensor t[7];
    float scale;
    void *out, *lse, *stream;
    if (!attention_views(a, t) || !number(a[7], scale)) return false;
    const Tensor& q = t[0];
    if (a[8] == Py_None || !buffer(a[8], at::kBFloat16, q.batch * q.tokens * q.heads * q.d, q.device, false, out) ||
        !buffer(a[9], at::kFloat, q.batch * q.heads * q.tokens, q.device, true, lse) || !current_stream(stream))
      return false;
    Py_BEGIN_ALLOW_THREADS
    status = apbv_host_attention(to_int(q.batch), to_int(q.heads), to_int(t[1].heads), to_int(q.d), q.view, t[1].view, t[2].view, t[3].view, t[4].view,
                                 t[5].view, t[6].view, scale, out, static_cast<float*>(lse), stream);
    Py_END_ALLOW_THREADS
    return true;
  });
}

// query_attention(seven tensors, scale, n_splits, out, lse_out, workspace)
PyObject* query_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 12) return not_taken();
  return guarded([&](int& status) {
    Tensor t[7];
    float scale;
    int64_t splits, ws_bytes;
    void *out, *lse, *ws, *stream;
    if (!attention_views(a, t) || !number(a[7], scale) || !whole(a[8], splits) || splits < -1 || splits > 0x7fffffff) return false;
    const Tensor& q = t[0];
    if (a[9] == Py_None || a[11] == Py_None || !buffer(a[9], at::kBFloat16, q.batch * q.tokens * q.heads * q.d, q.device, false, out) ||
        !buffer(a[10], at::kFloat, q.batch * q.heads * q.tokens, q.device, true, lse) ||
        !buffer(a[11], at::kByte, 0, q.device, false, ws, &ws_bytes) || !current_stream(stream))
      return false;
    Py_BEGIN_ALLOW_THREADS
    status = apbv_query_attention(to_int(q.batch), to_int(q.heads), to_int(t[1].heads), to_int(q.d), q.view, t[1].view, t[2].view, t[3].view, t[4].view,
                                  t[5].view, t[6].view, scale, (int)splits, out, static_cast<float*>(lse), ws, (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    return true;
  });
}

// attention_group(problems, scale, with_lse): every problem a tuple or list of seven tensors, out and (with_lse) lse_out
PyObject* attention_group(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3 || !(PyList_CheckExact(a[0]) || PyTuple_CheckExact(a[0])) || !PyBool_Check(a[2])) return not_taken();
  return guarded([&](int& status) {
    float scale;
    if (!number(a[1], scale)) return false;
    const Py_ssize_t count = PySequence_Fast_GET_SIZE(a[0]);
    if (count < 1 || count > 64) return false;
    std::vector<apbv_attention_item> items((size_t)count);
    int64_t hq = 0, hkv = 0, d = 0;
    for (Py_ssize_t m = 0; m < count; ++m) {
      PyObject* prob = PySequence_Fast_GET_ITEM(a[0], m);
      if (!(PyList_CheckExact(prob) || PyTuple_CheckExact(prob))) return false;
      const Py_ssize_t fields = PySequence_Fast_GET_SIZE(prob);
      PyObject** f = PySequence_Fast_ITEMS(prob);
      Tensor t[7];
      if (fields < 8 || fields > 9 || f[7] == Py_None || !attention_views(f, t, 3)) return false;
      PyObject* lse_obj = fields > 8 ? f[8] : Py_None;
      if (a[2] == Py_True && lse_obj == Py_None) return false;
      const Tensor& q = t[0];
      if (m == 0) {
        hq = q.heads;
        hkv = t[1].heads;
        d = q.d;
      } else if (q.heads != hq || t[1].heads != hkv || q.d != d) {
        return false;
      }
      void *out, *lse;
      if (!buffer(f[7], at::kBFloat16, q.tokens * hq * d, q.device, false, out) || !buffer(lse_obj, at::kFloat, hq * q.tokens, q.device, true, lse)) return false;
      apbv_attention_item& it = items[(size_t)m];
      it.q_local = q.view;
      it.k_anchor = t[1].view;
      it.v_anchor = t[2].view;
      it.k_pass = t[3].view;
      it.v_pass = t[4].view;
      it.k_local = t[5].view;
      it.v_local = t[6].view;
      it.out = out;
      it.lse_out = static_cast<float*>(lse);
    }
    void* stream;
    if (!current_stream(stream)) return false;
    Py_BEGIN_ALLOW_THREADS
    status = apbv_host_attention_group((int)count, items.data(), to_int(hq), to_int(hkv), to_int(d), scale, stream);
    Py_END_ALLOW_THREADS
    return true;
  });
}

// compress_kv(q_probe, k_local, v_local, l_p, reducer, scale, idx_out, k_c_out, v_c_out, scores_out, workspace);
// reducer: its number, or -1 for apbv_compress_kv_noalloc (workspace None)
PyObject* compress_kv(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 11) return not_taken();
  return guarded([&](int& status) {
    Tensor q, k, v;
    int64_t l_p, reducer, ws_bytes = 0;
    float scale;
    void *idx, *kc, *vc, *scores, *ws = nullptr, *stream;
    if (!view_of(a[0], q) || !view_of(a[1], k) || !view_of(a[2], v) || q.batch != k.batch || v.batch != k.batch) return false;
    if (!whole(a[3], l_p) || l_p < 0 || l_p > k.tokens || !whole(a[4], reducer) || !number(a[5], scale)) return false;
    const int64_t rows = k.batch * k.heads * l_p;
    if (a[6] == Py_None || a[7] == Py_None || a[8] == Py_None || !buffer(a[6], at::kInt, rows, k.device, false, idx) ||
        !buffer(a[7], at::kBFloat16, rows * q.d, k.device, false, kc) || !buffer(a[8], at::kBFloat16, rows * q.d, k.device, false, vc) ||
        !buffer(a[9], at::kDouble, k.batch * k.heads * k.tokens, k.device, true, scores))
      return false;
    if (reducer >= 0 && (a[10] == Py_None || !buffer(a[10], at::kByte, 0, k.device, false, ws, &ws_bytes))) return false;
    if (l_p == 0) idx = kc = vc = nullptr;
    if (!current_stream(stream)) return false;
    const int b = to_int(k.batch), hq = to_int(q.heads), hkv = to_int(k.heads), d = to_int(q.d);
    Py_BEGIN_ALLOW_THREADS
    if (reducer < 0)
      status = apbv_compress_kv_noalloc(b, hq, hkv, d, q.view, k.view, v.view, l_p, static_cast<int32_t*>(idx), kc, vc, static_cast<double*>(scores), stream);
    else if (reducer == APBV_REDUCE_SUM)
      status = apbv_compress_kv(b, hq, hkv, d, q.view, k.view, v.view, l_p, static_cast<int32_t*>(idx), kc, vc, static_cast<double*>(scores), ws, (size_t)ws_bytes, stream);
    else
      status = apbv_compress_kv_reduced((int)reducer, scale, b, hq, hkv, d, q.view, k.view, v.view, l_p, static_cast<int32_t*>(idx), kc, vc,
                                        static_cast<double*>(scores), ws, (size_t)ws_bytes, stream);
    Py_END_ALLOW_THREADS
    return true;
  });
}

// use_stream(is_initialized, current_device, raw_stream): the functions that name the current stream
PyObject* use_stream(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 3) {
    PyErr_SetString(PyExc_TypeError, "use_stream takes three functions");
    return nullptr;
  }
  PyObject** const kept[3] = {&g_is_initialized, &g_current_device, &g_raw_stream};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(a[i]);
    Py_XSETREF(*kept[i], a[i]);
  }
  Py_RETURN_NONE;
}

#define APBV_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {APBV_METHOD(merge_lse), APBV_METHOD(host_attention), APBV_METHOD(query_attention), APBV_METHOD(attention_group),
                         APBV_METHOD(compress_kv), APBV_METHOD(use_stream), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

// The module says what it was built against and linked to: the version of apbv.h, the address of the library's apbv_version.
PyMODINIT_FUNC PyInit__marshal() {
  PyObject* m = PyModule_Create(&module);
  PyObject* library = PyLong_FromVoidPtr(reinterpret_cast<void*>(&apbv_version));
  if (m == nullptr || library == nullptr || PyModule_AddIntConstant(m, "version", APBV_VERSION) != 0 || PyModule_AddObjectRef(m, "library", library) != 0)
    Py_CLEAR(m);
  Py_XDECREF(library);
  return m;
}
