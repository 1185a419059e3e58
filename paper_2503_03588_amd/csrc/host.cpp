// The calls of binding.py for the ordinary case, in one step from Python to the library: tensors that are plain, contiguous
// and on the GPU, the current stream.  Each function takes the arguments of the Python function of the same name, looks at
// them, allocates what the caller did not pass and calls the C entry point; it returns NotImplemented, having done nothing,
// whenever anything is out of the ordinary, and the Python function then goes its own way.  The library is called once: a
// status it reports is raised as the Python functions raise it.
//
// Reason: the smallest calls take 8 to 12 us on the GPU, and marshalling them in Python took 6 to 8 us each (tensor
// attributes, shapes, ctypes); now 3.5 to 5.  A list and a prefill of 1024 fp32 queries, two calls, were paced by it: 16.2 us
// -> 12.0; a call that is waited for: one decode step 21.7 -> 18.6 us, a chunk 46.3 -> 42.7, list and prefill 32.8 -> 25.6.
#include <algorithm>
#include <array>
#include <initializer_list>
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <c10/core/impl/LocalDispatchKeySet.h>
#include "../../include/powattn.h"

#ifndef POWATTN_HOST_DEVICE            // (the tests build this file for ordinary memory, where they stand in for the library)
#define POWATTN_HOST_DEVICE at::kCUDA
#endif

namespace {

// the library's entry points (addresses handed over by binding.py, which loads the library)
struct {
  decltype(&powattn_num_blocks) num_blocks;
  decltype(&powattn_max_k) max_k;
  decltype(&powattn_mask_build) mask_build;
  decltype(&powattn_prefill) prefill;
  decltype(&powattn_prefill_chunk) prefill_chunk;
  decltype(&powattn_prefill_chunk_paged) prefill_chunk_paged;
  decltype(&powattn_prefill_batch_paged) prefill_batch_paged;
  decltype(&powattn_prefill_varlen) prefill_varlen;
  decltype(&powattn_decode) decode;
  decltype(&powattn_decode_paged) decode_paged;
  decltype(&powattn_backward_workspace_bytes) backward_workspace_bytes;
  decltype(&powattn_backward) backward;
} lib;
PyObject* get_device = nullptr;       // torch._C._cuda_getDevice
PyObject* get_stream = nullptr;       // torch._C._cuda_getCurrentRawStream
PyObject* tensor_type = nullptr;      // torch.Tensor
PyObject* check = nullptr;            // binding._check: raises for a status

struct other_way {};                  // thrown: not the ordinary case
struct raised {};                     // thrown: the Python exception is set

void need(bool ok) { if (!ok) throw other_way{}; }

// plain tensors only: no subclass, no wrapper of a transform, nothing that a mode would want to see
const at::Tensor& tensor(PyObject* o) {
  need((PyObject*)Py_TYPE(o) == tensor_type);
  const at::Tensor& t = THPVariable_Unpack(o);
  need(t.defined() && t.device().type() == POWATTN_HOST_DEVICE && t.layout() == at::kStrided && t.is_contiguous());
  static const c10::DispatchKeySet wrappers({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::FuncTorchBatched,
                                             c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize,
                                             c10::DispatchKey::Conjugate, c10::DispatchKey::Negative, c10::DispatchKey::ZeroTensor});
  need(!t.key_set().has_any(wrappers));
  return t;
}
const at::Tensor& tensor_of(PyObject* o, at::ScalarType type, int64_t dims) {
  const at::Tensor& t = tensor(o);
  need(t.scalar_type() == type && t.dim() == dims);
  return t;
}
void* data(const at::Tensor& t) { return t.data_ptr(); }

int64_t whole(PyObject* o) {
  need(PyLong_CheckExact(o));
  const int64_t x = PyLong_AsLongLong(o);
  if (x == -1 && PyErr_Occurred()) { PyErr_Clear(); throw other_way{}; }
  return x;
}
float number(PyObject* o) {
  need(PyFloat_CheckExact(o));
  return (float)PyFloat_AS_DOUBLE(o);
}
powattn_pattern pattern(PyObject* values) {     // (block, window, sink, flags)
  need(PyTuple_CheckExact(values) && PyTuple_GET_SIZE(values) == 4);
  int64_t x[4];
  for (int i = 0; i < 4; ++i) {
    x[i] = whole(PyTuple_GET_ITEM(values, i));
    need(x[i] >= 0 && x[i] <= 0x7fffffff);
  }
  return {(int32_t)x[0], (int32_t)x[1], (int32_t)x[2], (uint32_t)x[3]};
}
void* current_stream() {
  PyObject* dev = PyObject_CallNoArgs(get_device);
  if (!dev) { PyErr_Clear(); throw other_way{}; }
  PyObject* s = PyObject_CallOneArg(get_stream, dev);
  Py_DECREF(dev);
  if (!s) { PyErr_Clear(); throw other_way{}; }
  void* p = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return p;
}
// no mode that wants to see the allocations below or the tensors
void no_modes() {
  need(!at::impl::torch_function_mode_enabled());
  const auto tls = c10::impl::tls_local_dispatch_key_set();
  need(!tls.included_.has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::PythonTLSSnapshot, c10::DispatchKey::Functionalize,
                                                  c10::DispatchKey::FuncTorchBatched, c10::DispatchKey::FuncTorchDynamicLayerFrontMode})));
}
int32_t dtype_code(const at::Tensor& t) {
  if (t.scalar_type() == at::kBFloat16) return POWATTN_BF16;
  need(t.scalar_type() == at::kFloat);
  return POWATTN_F32;
}
// Other Python threads run while it lives, as in torch's own allocations (one that waits for the GPU may wait for a callback
// that needs the interpreter).  The interpreter is this thread's again whichever way the scope is left: the outputs are
// allocated and the library's arguments formed inside it, and both throw.
struct without_gil {
  PyThreadState* ts = PyEval_SaveThread();
  ~without_gil() { PyEval_RestoreThread(ts); }
};
// the allocations and the library's call, `name` being its entry point
template <class F>
void call(const char* name, F&& f) {
  void* stream = current_stream();
  int st;
  {
    without_gil others_run;
    st = f(stream);
  }
  if (st == POWATTN_OK) return;
  // (not other_way: the Python way would call again, and a HIP error is reported once: the second call would launch)
  PyObject* r = PyObject_CallFunction(check, "is", st, name);
  if (r) {
    Py_DECREF(r);
    PyErr_Format(PyExc_RuntimeError, "%s: status %d", name, st);
  }
  throw raised{};
}
int32_t small(int64_t x) { need(x >= 0 && x <= 0x7fffffff); return (int32_t)x; }

// o and lse: the caller's, or new ones (allocate(), with other threads running); returned as the pair that the Python
// functions return
struct outputs {
  PyObject* o_arg; PyObject* lse_arg;
  const at::Tensor& q;
  std::array<int64_t, 3> lse_shape;
  size_t lse_dims;
  bool new_lse, zeros;
  at::Tensor o, lse;
  outputs(PyObject* o_in, PyObject* lse_in, PyObject* want_lse, const at::Tensor& queries, std::initializer_list<int64_t> shape,
          bool zeroed = false)
      : o_arg(o_in), lse_arg(lse_in), q(queries), lse_dims(shape.size()), zeros(zeroed) {
    need(want_lse == Py_True || want_lse == Py_False);
    std::copy(shape.begin(), shape.end(), lse_shape.begin());
    if (o_arg != Py_None) o = tensor(o_arg);
    if (lse_arg != Py_None) lse = tensor(lse_arg);
    new_lse = lse_arg == Py_None && want_lse == Py_True;
  }
  void allocate() {
    if (o_arg == Py_None) o = zeros ? at::zeros_like(q) : at::empty_like(q);
    if (new_lse) {
      const auto opt = q.options().dtype(at::kFloat);
      const at::IntArrayRef shape(lse_shape.data(), lse_dims);
      lse = zeros ? at::zeros(shape, opt) : at::empty(shape, opt);
    }
  }
  float* lse_ptr() { return lse.defined() ? (float*)data(lse) : nullptr; }
  PyObject* pair() {
    PyObject* t = PyTuple_New(2);
    if (!t) return nullptr;
    if (o_arg != Py_None) { Py_INCREF(o_arg); PyTuple_SET_ITEM(t, 0, o_arg); } else PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(o));
    if (lse_arg != Py_None) { Py_INCREF(lse_arg); PyTuple_SET_ITEM(t, 1, lse_arg); }
    else if (lse.defined()) PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(lse));
    else { Py_INCREF(Py_None); PyTuple_SET_ITEM(t, 1, Py_None); }
    return t;
  }
};
struct lists {
  const int32_t* cnt = nullptr; const int32_t* idx = nullptr;
  int32_t max_k = 0;
  int64_t rows = 0;
  bool given;
  lists(PyObject* c, PyObject* i) : given(i != Py_None) {
    need((c == Py_None) == (i == Py_None));
    if (!given) return;
    const at::Tensor& tc = tensor_of(c, at::kInt, 1);
    const at::Tensor& ti = tensor_of(i, at::kInt, 2);
    cnt = (const int32_t*)data(tc); idx = (const int32_t*)data(ti);
    max_k = small(ti.size(1));
    rows = tc.size(0);
  }
};
struct pages {                         // [n_pages, hkv, block, d] twice, and the table [batch, stride]
  const void* k; const void* v; const int32_t* table;
  int64_t n; int32_t hkv, stride;
  pages(PyObject* ko, PyObject* vo, PyObject* to, const powattn_pattern& pat, int64_t batch, int64_t d, at::ScalarType type) {
    const at::Tensor& tk = tensor_of(ko, type, 4);
    const at::Tensor& tv = tensor_of(vo, type, 4);
    const at::Tensor& tt = tensor_of(to, at::kInt, 2);
    need(tk.sizes() == tv.sizes() && tk.size(2) == pat.block && tk.size(3) == d && tt.size(0) == batch);
    k = data(tk); v = data(tv); table = (const int32_t*)data(tt);
    n = tk.size(0); hkv = small(tk.size(1)); stride = small(tt.size(1));
  }
};

template <class F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t expected, F&& f) {
  if (n != expected) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
  try {
    no_modes();
    PyObject* r = f();
    if (r) return r;
    PyErr_Clear();
  } catch (const raised&) {
    return nullptr;
  } catch (const other_way&) {
  } catch (const std::exception&) {    // (an allocation that failed: the Python way raises it)
  }
  Py_INCREF(Py_NotImplemented);
  return Py_NotImplemented;
}

PyObject* f_mask_build(PyObject*, PyObject* const* a, Py_ssize_t n) {   // values, seq_len
  return guarded(n, 2, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const int64_t len = whole(a[1]);
    const int64_t nb = lib.num_blocks(&pat, len);
    const int32_t mk = lib.max_k(&pat, len);
    need(nb > 0 && mk > 0);
    const auto opt = at::TensorOptions().dtype(at::kInt).device(POWATTN_HOST_DEVICE);
    at::Tensor idx, cnt;
    call("powattn_mask_build", [&](void* stream) {
      idx = at::empty({nb, (int64_t)mk}, opt);
      cnt = at::empty({nb}, opt);
      return lib.mask_build(&pat, len, (int32_t*)data(cnt), (int32_t*)data(idx), mk, nullptr, stream);
    });
    PyObject* t = PyTuple_New(3);
    if (!t) return nullptr;
    PyTuple_SET_ITEM(t, 0, THPVariable_Wrap(cnt));
    PyTuple_SET_ITEM(t, 1, THPVariable_Wrap(idx));
    Py_INCREF(Py_None);
    PyTuple_SET_ITEM(t, 2, Py_None);
    return t;
  });
}
// values, kv_cnt, kv_idx, q, k, v, o, lse, softmax_scale, want_lse
PyObject* f_prefill(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4);
    const int64_t b = q.size(0), hq = q.size(1), len = q.size(2), d = q.size(3);
    const at::Tensor& k = tensor_of(a[4], q.scalar_type(), 4);
    const at::Tensor& v = tensor_of(a[5], q.scalar_type(), 4);
    need(k.sizes() == v.sizes() && k.size(0) == b && k.size(2) == len && k.size(3) == d);
    need(!l.given || l.rows * pat.block >= len);
    const int32_t code = dtype_code(q);
    const float scale = number(a[8]);
    outputs out(a[6], a[7], a[9], q, {b, hq, len});
    call("powattn_prefill", [&](void* stream) { out.allocate(); return lib.prefill(&pat, l.cnt, l.idx, l.max_k, data(q), data(k), data(v), data(out.o), out.lse_ptr(), small(b), small(hq),
                     small(k.size(1)), len, small(d), code, scale, stream); });
    return out.pair();
  });
}
// values, kv_cnt, kv_idx, q, k_cache, v_cache, q_start, o, lse, softmax_scale, want_lse
PyObject* f_prefill_chunk(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4);
    const int64_t b = q.size(0), hq = q.size(1), len = q.size(2), d = q.size(3), start = whole(a[6]);
    const at::Tensor& k = tensor_of(a[4], q.scalar_type(), 4);
    const at::Tensor& v = tensor_of(a[5], q.scalar_type(), 4);
    need(k.sizes() == v.sizes() && k.size(0) == b && k.size(3) == d);
    need(!l.given || l.rows * pat.block >= start + len);
    const int32_t code = dtype_code(q);
    const float scale = number(a[9]);
    outputs out(a[7], a[8], a[10], q, {b, hq, len});
    call("powattn_prefill_chunk", [&](void* stream) { out.allocate(); return lib.prefill_chunk(&pat, l.cnt, l.idx, l.max_k, data(q), data(k), data(v), data(out.o), out.lse_ptr(), small(b), small(hq),
                           small(k.size(1)), start, len, k.size(2), small(d), code, scale, stream); });
    return out.pair();
  });
}
// values, kv_cnt, kv_idx, q, k_pages, v_pages, block_table, q_start, o, lse, softmax_scale, want_lse
PyObject* f_prefill_chunk_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4 && l.given);
    const int64_t b = q.size(0), hq = q.size(1), len = q.size(2), d = q.size(3), start = whole(a[7]);
    const pages pg(a[4], a[5], a[6], pat, b, d, q.scalar_type());
    need(l.rows * pat.block >= start + len);
    const int32_t code = dtype_code(q);
    const float scale = number(a[10]);
    outputs out(a[8], a[9], a[11], q, {b, hq, len});
    call("powattn_prefill_chunk_paged", [&](void* stream) { out.allocate(); return lib.prefill_chunk_paged(&pat, l.cnt, l.idx, l.max_k, data(q), pg.k, pg.v, pg.table, pg.stride, pg.n, data(out.o), out.lse_ptr(),
                                 small(b), small(hq), pg.hkv, start, len, small(d), code, scale, stream); });
    return out.pair();
  });
}
// values, kv_cnt, kv_idx, q, k_pages, v_pages, block_table, q_start, q_len, o, lse, softmax_scale, want_lse
PyObject* f_prefill_batch_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 13, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4 && l.given);
    const int64_t b = q.size(0), hq = q.size(1), rows = q.size(2), d = q.size(3);
    const pages pg(a[4], a[5], a[6], pat, b, d, q.scalar_type());
    const at::Tensor& start = tensor_of(a[7], at::kInt, 1);
    const at::Tensor& len = tensor_of(a[8], at::kInt, 1);
    need(start.size(0) == b && len.size(0) == b && start.device() == q.device() && len.device() == q.device() && l.rows >= pg.stride);
    const int32_t code = dtype_code(q);
    const float scale = number(a[11]);
    outputs out(a[9], a[10], a[12], q, {b, hq, rows});
    call("powattn_prefill_batch_paged", [&](void* stream) { out.allocate(); return lib.prefill_batch_paged(&pat, l.cnt, l.idx, l.max_k, data(q), pg.k, pg.v, pg.table, pg.stride, pg.n, (const int32_t*)data(start),
                                 (const int32_t*)data(len), rows, data(out.o), out.lse_ptr(), small(b), small(hq), pg.hkv, small(d),
                                 code, scale, stream); });
    return out.pair();
  });
}
// values, kv_cnt, kv_idx, q, k, v, seq_lens, o, lse, softmax_scale, want_lse
PyObject* f_prefill_varlen(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4);
    const int64_t b = q.size(0), hq = q.size(1), len = q.size(2), d = q.size(3);
    const at::Tensor& k = tensor_of(a[4], q.scalar_type(), 4);
    const at::Tensor& v = tensor_of(a[5], q.scalar_type(), 4);
    const at::Tensor& lens = tensor_of(a[6], at::kInt, 1);
    need(k.sizes() == v.sizes() && k.size(0) == b && k.size(2) == len && k.size(3) == d && lens.size(0) == b && lens.device() == q.device());
    need(!l.given || l.rows * pat.block >= len);
    const int32_t code = dtype_code(q);
    const float scale = number(a[9]);
    outputs out(a[7], a[8], a[10], q, {b, hq, len}, true);
    call("powattn_prefill_varlen", [&](void* stream) { out.allocate(); return lib.prefill_varlen(&pat, l.cnt, l.idx, l.max_k, data(q), data(k), data(v), data(out.o), out.lse_ptr(), small(b), small(hq),
                            small(k.size(1)), (const int32_t*)data(lens), len, small(d), code, scale, stream); });
    return out.pair();
  });
}
// values, q, k_cache, v_cache, kv_len, o, lse, softmax_scale, workspace, want_lse
PyObject* f_decode(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 10, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const at::Tensor& q = tensor(a[1]);
    need(q.dim() == 3);
    const int64_t b = q.size(0), hq = q.size(1), d = q.size(2);
    const at::Tensor& k = tensor_of(a[2], q.scalar_type(), 4);
    const at::Tensor& v = tensor_of(a[3], q.scalar_type(), 4);
    const at::Tensor& lens = tensor_of(a[4], at::kInt, 1);
    need(k.sizes() == v.sizes() && k.size(0) == b && k.size(3) == d && lens.size(0) == b);
    const at::Tensor& ws = tensor(a[8]);
    const int32_t code = dtype_code(q);
    const float scale = number(a[7]);
    outputs out(a[5], a[6], a[9], q, {b, hq});
    call("powattn_decode", [&](void* stream) { out.allocate(); return lib.decode(&pat, data(q), data(k), data(v), (const int32_t*)data(lens), k.size(2), data(out.o), out.lse_ptr(), small(b), small(hq),
                    small(k.size(1)), small(d), code, scale, data(ws), ws.nbytes(), stream); });
    return out.pair();
  });
}
// values, q, k_pages, v_pages, block_table, kv_len, o, lse, softmax_scale, workspace, want_lse
PyObject* f_decode_paged(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const at::Tensor& q = tensor(a[1]);
    need(q.dim() == 3);
    const int64_t b = q.size(0), hq = q.size(1), d = q.size(2);
    const pages pg(a[2], a[3], a[4], pat, b, d, q.scalar_type());
    const at::Tensor& lens = tensor_of(a[5], at::kInt, 1);
    need(lens.size(0) == b);
    const at::Tensor& ws = tensor(a[9]);
    const int32_t code = dtype_code(q);
    const float scale = number(a[8]);
    outputs out(a[6], a[7], a[10], q, {b, hq});
    call("powattn_decode_paged", [&](void* stream) { out.allocate(); return lib.decode_paged(&pat, data(q), pg.k, pg.v, pg.n, pg.table, pg.stride, (const int32_t*)data(lens), data(out.o), out.lse_ptr(),
                          small(b), small(hq), pg.hkv, small(d), code, scale, data(ws), ws.nbytes(), stream); });
    return out.pair();
  });
}

// values, kv_cnt, kv_idx, q, k, v, o, lse, d_o, dq, dk, dv, softmax_scale, workspace
PyObject* f_backward(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 14, [&]() -> PyObject* {
    const powattn_pattern pat = pattern(a[0]);
    const lists l(a[1], a[2]);
    const at::Tensor& q = tensor(a[3]);
    need(q.dim() == 4 && l.given);
    const int64_t b = q.size(0), hq = q.size(1), len = q.size(2), d = q.size(3);
    const at::ScalarType type = q.scalar_type();
    const at::Tensor& k = tensor_of(a[4], type, 4);
    const at::Tensor& v = tensor_of(a[5], type, 4);
    const at::Tensor& o = tensor_of(a[6], type, 4);
    const at::Tensor& lse = tensor_of(a[7], at::kFloat, 3);
    const at::Tensor& dout = tensor_of(a[8], type, 4);
    need(k.sizes() == v.sizes() && k.size(0) == b && k.size(2) == len && k.size(3) == d && o.sizes() == q.sizes() && dout.sizes() == q.sizes()
         && lse.size(0) == b && lse.size(1) == hq && lse.size(2) == len);
    const int32_t code = dtype_code(q), hkv = small(k.size(1));
    const float scale = number(a[12]);
    const at::Tensor* like[3] = {&q, &k, &v};
    at::Tensor grad[3], ws;
    for (int i = 0; i < 3; ++i) if (a[9 + i] != Py_None) grad[i] = tensor(a[9 + i]);
    if (a[13] != Py_None) ws = tensor(a[13]);
    size_t bytes = 0;
    if (!ws.defined()) {
      bytes = lib.backward_workspace_bytes(&pat, small(b), small(hq), hkv, len, small(d));
      need(bytes > 0);
    }
    call("powattn_backward", [&](void* stream) {
      for (int i = 0; i < 3; ++i) if (!grad[i].defined()) grad[i] = at::empty_like(*like[i]);
      if (!ws.defined()) ws = at::empty({(int64_t)bytes}, q.options().dtype(at::kByte));
      return lib.backward(&pat, l.cnt, l.idx, l.max_k, data(q), data(k), data(v), data(o), (const float*)data(lse), data(dout),
                          data(grad[0]), data(grad[1]), data(grad[2]), small(b), small(hq), hkv, len, small(d), code,
                          scale, data(ws), ws.nbytes(), stream);
    });
    PyObject* t = PyTuple_New(3);
    if (!t) return nullptr;
    for (int i = 0; i < 3; ++i) {
      if (a[9 + i] != Py_None) { Py_INCREF(a[9 + i]); PyTuple_SET_ITEM(t, i, a[9 + i]); }
      else PyTuple_SET_ITEM(t, i, THPVariable_Wrap(grad[i]));
    }
    return t;
  });
}

// addresses of the entry points in the order of `lib`, torch.Tensor, the device and the stream look-up, binding._check
PyObject* f_bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr Py_ssize_t N_FN = sizeof(lib) / sizeof(void*);
  if (n != N_FN + 4) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
  void* fn[N_FN];
  for (Py_ssize_t i = 0; i < N_FN; ++i) {
    fn[i] = PyLong_AsVoidPtr(a[i]);
    if (!fn[i]) { if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null entry point"); return nullptr; }
  }
  memcpy(&lib, fn, sizeof lib);
  for (int i = 0; i < 4; ++i) Py_INCREF(a[N_FN + i]);
  tensor_type = a[N_FN]; get_device = a[N_FN + 1]; get_stream = a[N_FN + 2]; check = a[N_FN + 3];
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)())f_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {FAST(bind), FAST(mask_build), FAST(prefill), FAST(prefill_chunk), FAST(prefill_chunk_paged), FAST(prefill_batch_paged),
                         FAST(prefill_varlen), FAST(decode), FAST(decode_paged), FAST(backward), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() { return PyModule_Create(&module); }
