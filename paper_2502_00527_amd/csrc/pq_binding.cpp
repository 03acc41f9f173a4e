// Argument marshalling of the calls a serving loop makes, as a CPython extension: tensors to device pointers and
// sizes, and the call of the C entry point.  The checks are those of the Python functions of the same names in
// __init__.py, and a call that does not pass all of them is not made: the function returns None, and the
// Python function goes through its own checks, which raise with a message, or handle what is unusual (an
// integer that is no int, a tensor subclass).  Otherwise the entry point's status is returned.
//
// Why it is native: read through Python attributes and ctypes the arguments of a decode call took 12 us, which
// is as long as the whole kernel of a short context.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <climits>
#include <cstring>

#include "polarquant.h"

namespace {

// The value of an argument that is not usable here; unwinds to the function's end, which returns None.
struct Decline {};

// The layout class of __init__.py; no other object is taken for a layout, whatever bytes it holds.
PyObject* layout_type = nullptr;
pq_layout layout_of(PyObject* o) {
  Py_buffer buffer;
  if (!layout_type || reinterpret_cast<PyObject*>(Py_TYPE(o)) != layout_type || PyObject_GetBuffer(o, &buffer, PyBUF_SIMPLE) != 0) throw Decline{};
  pq_layout layout;
  const bool whole = buffer.len == static_cast<Py_ssize_t>(sizeof(layout));
  if (whole) memcpy(&layout, buffer.buf, sizeof(layout));
  PyBuffer_Release(&buffer);
  if (!whole) throw Decline{};
  return layout;
}

const at::Tensor& device_tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw Decline{};
  const at::Tensor& t = THPVariable_Unpack(o);
  // plain strided memory: no wrapper of a transform, no fake or lazy tensor
  if (!t.defined() || !t.is_cuda() || t.layout() != c10::kStrided || !t.has_storage() ||
      t.key_set().has_any(c10::DispatchKeySet({c10::DispatchKey::Python, c10::DispatchKey::FuncTorchBatched,
                                               c10::DispatchKey::FuncTorchGradWrapper, c10::DispatchKey::Functionalize})))
    throw Decline{};
  return t;
}
const at::Tensor& contiguous_tensor(PyObject* o) {
  const at::Tensor& t = device_tensor(o);
  if (!t.is_contiguous()) throw Decline{};
  return t;
}
const at::Tensor& contiguous_tensor(PyObject* o, at::ScalarType type) {
  const at::Tensor& t = contiguous_tensor(o);
  if (t.scalar_type() != type) throw Decline{};
  return t;
}
pq_dtype float_kind(const at::Tensor& t) {
  if (t.scalar_type() == at::kHalf) return PQ_F16;
  if (t.scalar_type() == at::kFloat) return PQ_F32;
  throw Decline{};
}
size_t bytes_of(const at::Tensor& t) { return static_cast<size_t>(t.numel()) * t.element_size(); }
int64_t integer(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw Decline{};
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow) throw Decline{};
  return v;
}
int32_t integer32(int64_t v) {
  if (v < INT_MIN || v > INT_MAX) throw Decline{};
  return static_cast<int32_t>(v);
}

// torch's current stream on its current device, as a hipStream_t
PyObject *get_device = nullptr, *get_raw_stream = nullptr;
void* current_stream() {
  if (!get_device || !get_raw_stream) throw Decline{};
  PyObject* const device = PyObject_CallNoArgs(get_device);
  if (!device) throw Decline{};
  PyObject* const stream = PyObject_CallOneArg(get_raw_stream, device);
  Py_DECREF(device);
  if (!stream) throw Decline{};
  void* const p = PyLong_AsVoidPtr(stream);
  Py_DECREF(stream);
  if (!p && PyErr_Occurred()) throw Decline{};
  return p;
}
int64_t pages(size_t bytes, size_t page) { return static_cast<int64_t>(bytes / (page > 0 ? page : 1)); }

// Pages the codes pool holds; the parameter pool holds as many.
int64_t key_pool_pages(const pq_layout* l, const at::Tensor& codes, const at::Tensor& params) {
  const int64_t n = pages(bytes_of(codes), pq_codes_bytes_per_page(l));
  if (bytes_of(params) < static_cast<size_t>(n) * pq_params_bytes_per_page(l)) throw Decline{};
  return n;
}
void check_rows(const at::Tensor& t, const pq_layout* l, bool heads) {
  if (t.dim() != 3 || t.size(2) != l->head_dim || (heads && t.size(1) != l->n_kv_heads)) throw Decline{};
}

// Runs `call`, which returns a status; None if it declines.  The entry points are called without the interpreter lock.
template <typename F>
PyObject* guarded(Py_ssize_t n_args, Py_ssize_t want, F call) {
  if (n_args != want) Py_RETURN_NONE;
  try {
    return PyLong_FromLong(call());
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename F>
int without_lock(F f) {
  const Unlocked unlocked;
  return f();
}

// (layout, q, codes, params, v_pool, block_table, seq_lens, max_seq_len, sm_scale, out, workspace, scores, residual,
//  v_bits, v_params)
PyObject* decode_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 15, [&] {
    const pq_layout layout = layout_of(a[0]), *const l = &layout;
    const at::Tensor& q = contiguous_tensor(a[1]);
    check_rows(q, l, false);
    const at::Tensor &codes = contiguous_tensor(a[2]), &params = contiguous_tensor(a[3]);
    const int64_t n_pages = key_pool_pages(l, codes, params);
    const int32_t v_bits = integer32(integer(a[13]));
    const at::Tensor& v = contiguous_tensor(a[4], v_bits == 16 ? at::kHalf : at::kByte);
    void* v_params = nullptr;
    int64_t v_pages;
    if (v_bits == 16) {
      v_pages = pages(bytes_of(v), pq_values_bytes_per_page(l));
    } else {
      v_params = contiguous_tensor(a[14], at::kHalf).data_ptr();
      v_pages = pages(bytes_of(v), pq_vq_bytes_per_page(l, v_bits));
    }
    if (v_pages < n_pages) throw Decline{};
    const at::Tensor &table = contiguous_tensor(a[5], at::kInt), &lens = contiguous_tensor(a[6], at::kInt);
    if (table.dim() < 2) throw Decline{};
    const int32_t max_seq_len = integer32(integer(a[7]));
    if (!PyFloat_CheckExact(a[8])) throw Decline{};
    const float sm_scale = static_cast<float>(PyFloat_AS_DOUBLE(a[8]));
    const at::Tensor &out = contiguous_tensor(a[9], at::kFloat), &workspace = contiguous_tensor(a[10]);
    float* scores = nullptr;
    int64_t scores_stride = 0;
    if (a[11] != Py_None) {
      const at::Tensor& s = contiguous_tensor(a[11], at::kFloat);
      if (s.dim() < 1) throw Decline{};
      scores = static_cast<float*>(s.data_ptr());
      scores_stride = s.size(-1);
    }
    void* const residual = a[12] == Py_None ? nullptr : contiguous_tensor(a[12], at::kHalf).data_ptr();
    const int32_t n_seqs = integer32(q.size(0)), n_heads = integer32(q.size(1)), width = integer32(table.size(1));
    const pq_dtype kind = float_kind(q);
    void *const qp = q.data_ptr(), *const cp = codes.data_ptr(), *const pp = params.data_ptr(), *const vp = v.data_ptr(),
         *const ws = workspace.data_ptr(), *const stream = current_stream();
    const int32_t *const tp = static_cast<const int32_t*>(table.data_ptr()), *const lp = static_cast<const int32_t*>(lens.data_ptr());
    float* const op = static_cast<float*>(out.data_ptr());
    const size_t ws_bytes = bytes_of(workspace);
    return without_lock([&] {
      return pq_decode_attention(l, qp, kind, n_seqs, n_heads, cp, pp, vp, v_bits, v_params, n_pages, tp, width, lp,
                                 max_seq_len, sm_scale, op, scores, scores_stride, residual, ws, ws_bytes, stream);
    });
  });
}

// (layout, q, codes, params, block_table, seq_lens, max_seq_len, scores, residual)
PyObject* score_keys(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&] {
    const pq_layout layout = layout_of(a[0]), *const l = &layout;
    const at::Tensor& q = contiguous_tensor(a[1]);
    check_rows(q, l, false);
    const at::Tensor &codes = contiguous_tensor(a[2]), &params = contiguous_tensor(a[3]);
    const int64_t n_pages = key_pool_pages(l, codes, params);
    const at::Tensor &table = contiguous_tensor(a[4], at::kInt), &lens = contiguous_tensor(a[5], at::kInt);
    if (table.dim() < 2) throw Decline{};
    const int32_t max_seq_len = integer32(integer(a[6]));
    const at::Tensor& s = contiguous_tensor(a[7], at::kFloat);
    if (s.dim() < 1) throw Decline{};
    void* const residual = a[8] == Py_None ? nullptr : contiguous_tensor(a[8], at::kHalf).data_ptr();
    const int32_t n_seqs = integer32(q.size(0)), n_heads = integer32(q.size(1)), width = integer32(table.size(1));
    const pq_dtype kind = float_kind(q);
    void *const qp = q.data_ptr(), *const cp = codes.data_ptr(), *const pp = params.data_ptr(), *const stream = current_stream();
    const int32_t *const tp = static_cast<const int32_t*>(table.data_ptr()), *const lp = static_cast<const int32_t*>(lens.data_ptr());
    float* const sp = static_cast<float*>(s.data_ptr());
    const int64_t stride = s.size(-1);
    return without_lock([&] {
      return pq_score_keys(l, qp, kind, n_seqs, n_heads, cp, pp, n_pages, tp, width, lp, max_seq_len, sp, stride, residual, stream);
    });
  });
}

// (layout, keys, page_ids, codes, params)
PyObject* encode_keys(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 5, [&] {
    const pq_layout layout = layout_of(a[0]), *const l = &layout;
    const at::Tensor& keys = device_tensor(a[1]);
    check_rows(keys, l, true);
    if (keys.stride(2) != 1) throw Decline{};
    const at::Tensor &codes = contiguous_tensor(a[3]), &params = contiguous_tensor(a[4]);
    const int64_t n_pages = key_pool_pages(l, codes, params);
    const pq_dtype kind = float_kind(keys);
    const int32_t* const ids = static_cast<const int32_t*>(contiguous_tensor(a[2], at::kInt).data_ptr());
    void *const kp = keys.data_ptr(), *const cp = codes.data_ptr(), *const pp = params.data_ptr(), *const stream = current_stream();
    const int64_t token_stride = keys.stride(0), head_stride = keys.stride(1), tokens = keys.size(0);
    return without_lock([&] { return pq_encode_keys(l, kp, kind, token_stride, head_stride, tokens, ids, cp, pp, n_pages, stream); });
  });
}

// (layout, v_bits, values, page_ids, vq_pool, vq_params)
PyObject* encode_values(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&] {
    const pq_layout layout = layout_of(a[0]), *const l = &layout;
    const int32_t v_bits = integer32(integer(a[1]));
    const at::Tensor& values = device_tensor(a[2]);
    check_rows(values, l, true);
    if (values.scalar_type() != at::kHalf || values.stride(2) != 1) throw Decline{};
    const int32_t* const ids = static_cast<const int32_t*>(contiguous_tensor(a[3], at::kInt).data_ptr());
    const at::Tensor &pool = contiguous_tensor(a[4], at::kByte), &params = contiguous_tensor(a[5], at::kHalf);
    const int64_t n_pages = pages(bytes_of(pool), pq_vq_bytes_per_page(l, v_bits));
    void *const vp = values.data_ptr(), *const qp = pool.data_ptr(), *const pp = params.data_ptr(), *const stream = current_stream();
    const int64_t token_stride = values.stride(0), head_stride = values.stride(1), tokens = values.size(0);
    return without_lock([&] { return pq_encode_values(l, v_bits, vp, token_stride, head_stride, tokens, ids, qp, pp, n_pages, stream); });
  });
}

// (layout, new_keys, residual, seq_lens, block_table, codes, params)
PyObject* append_keys(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&] {
    const pq_layout layout = layout_of(a[0]), *const l = &layout;
    const at::Tensor& keys = contiguous_tensor(a[1]);
    check_rows(keys, l, true);
    const at::Tensor &codes = contiguous_tensor(a[5]), &params = contiguous_tensor(a[6]);
    const int64_t n_pages = key_pool_pages(l, codes, params);
    const pq_dtype kind = float_kind(keys);
    void* const residual = contiguous_tensor(a[2], at::kHalf).data_ptr();
    const at::Tensor &lens = contiguous_tensor(a[3], at::kInt), &table = contiguous_tensor(a[4], at::kInt);
    if (table.dim() < 2) throw Decline{};
    const int32_t n_seqs = integer32(keys.size(0)), width = integer32(table.size(1));
    void *const kp = keys.data_ptr(), *const cp = codes.data_ptr(), *const pp = params.data_ptr(), *const stream = current_stream();
    const int32_t *const tp = static_cast<const int32_t*>(table.data_ptr()), *const lp = static_cast<const int32_t*>(lens.data_ptr());
    return without_lock([&] { return pq_append_keys(l, kp, kind, n_seqs, residual, lp, tp, width, cp, pp, n_pages, stream); });
  });
}

PyObject* set_layout_type(PyObject*, PyObject* type) {
  Py_INCREF(type);
  Py_XSETREF(layout_type, type);
  Py_RETURN_NONE;
}

#define PQ_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {PQ_METHOD(decode_attention), PQ_METHOD(score_keys), PQ_METHOD(encode_keys), PQ_METHOD(encode_values),
                         PQ_METHOD(append_keys), {"set_layout_type", set_layout_type, METH_O, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_native", "Argument marshalling for libpolarquant.", -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) {
  // tensors are read through the headers of one torch
  PyObject* const torch = PyImport_ImportModule("torch");
  if (!torch) return nullptr;
  PyObject* const version = PyObject_GetAttrString(torch, "__version__");
  Py_DECREF(torch);
  if (!version) return nullptr;
  PyObject* const text = PyObject_Str(version);
  Py_DECREF(version);
  if (!text) return nullptr;
  const bool same = PyUnicode_CompareWithASCIIString(text, PQ_TORCH_VERSION) == 0;
  if (!same) PyErr_Format(PyExc_ImportError, "_native was built for torch %s, this is %U", PQ_TORCH_VERSION, text);
  Py_DECREF(text);
  if (!same) return nullptr;
  PyObject* const torch_c = PyImport_ImportModule("torch._C");
  if (!torch_c) return nullptr;
  get_device = PyObject_GetAttrString(torch_c, "_cuda_getDevice");
  get_raw_stream = PyObject_GetAttrString(torch_c, "_cuda_getCurrentRawStream");
  PyErr_Clear();                                  // a torch without devices: every call declines
  Py_DECREF(torch_c);
  return PyModule_Create(&module);
}
