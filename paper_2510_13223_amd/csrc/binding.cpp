// binding.cpp -- native argument checks of the Python binding (a CPython extension, host code only).
//
// A call through the Python binding checks some ten tensors (type, device, dtype, contiguity, shape)
// and builds the C ABI's arguments.  Written in Python that took about 17 us of a call, more than the
// whole device time of a short one.  Each function here makes the same checks and calls the C ABI;
// it returns the call's status, or None where anything is not as the checks want it (or not a plain
// tensor): the Python binding then runs its own checks, which say what is wrong.  Nothing is kept
// from one call for the next but the addresses of the C ABI.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/core/impl/DeviceGuardImplInterface.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstring>
#include <initializer_list>

#include "bana.h"

namespace {

struct Api {
  decltype(&bana_decode_attn_partial) partial;
  decltype(&bana_decode_attn_partial_noalloc) noalloc;
  decltype(&bana_decode_attn_fused) fused;
  decltype(&bana_decode_attn_fused_copies) fused_copies;
  decltype(&bana_decode_attn_heads) heads;
  decltype(&bana_merge_partials) merge;
  decltype(&bana_migrate_kv_blocks) migrate;
};
Api g_api{};
PyObject* g_raw_stream = nullptr;  // torch._C._cuda_getCurrentRawStream
PyObject* g_stream_type = nullptr; // torch.cuda.Stream
PyObject* g_dims_type = nullptr;   // the ctypes bana_dims

constexpr int kMaxCopies = 16;  // more than the C ABI takes; longer lists go the Python way

// The tensors of one call: wanted ones, all on one device.
struct Args {
  int device = -1;

  // Tensor `o` as wanted, or nullptr.
  const at::Tensor* get(PyObject* o, at::ScalarType dtype) {
    const at::Tensor* t = any(o);
    return t != nullptr && t->scalar_type() == dtype ? t : nullptr;
  }
  const at::Tensor* get(PyObject* o, at::ScalarType dtype, std::initializer_list<int64_t> shape) {
    const at::Tensor* t = get(o, dtype);
    return t != nullptr && t->sizes() == at::IntArrayRef(shape.begin(), shape.size()) ? t : nullptr;
  }
  // A contiguous device tensor of any type.
  const at::Tensor* any(PyObject* o) {
    if (!THPVariable_CheckExact(o)) return nullptr;
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) return nullptr;
    const int d = t.get_device();
    if (device < 0) device = d;
    return d == device ? &t : nullptr;
  }
  bool on_current_device() const {
    return c10::impl::getDeviceGuardImpl(c10::DeviceType::CUDA)->getDevice().index() == device;
  }
};

// The stream handle of a call: an int, a stream object, or None for the current stream.
bool stream_handle(PyObject* o, int device, void** out) {
  PyObject* h;
  if (o == Py_None) {
    PyObject* index = PyLong_FromLong(device);
    if (index == nullptr) return false;
    h = PyObject_CallOneArg(g_raw_stream, index);
    Py_DECREF(index);
  } else if (PyLong_CheckExact(o)) {
    Py_INCREF(o);
    h = o;
  } else {
    if (PyObject_IsInstance(o, g_stream_type) != 1) return false;
    h = PyObject_GetAttrString(o, "cuda_stream");
  }
  if (h == nullptr) return false;
  *out = PyLong_AsVoidPtr(h);
  Py_DECREF(h);
  return !PyErr_Occurred();
}

bool int_arg(PyObject* o, long long* out) {
  if (!PyLong_CheckExact(o)) return false;
  *out = PyLong_AsLongLong(o);
  return !PyErr_Occurred();
}

template <typename T>
T* data(const at::Tensor* t) {
  return t == nullptr ? nullptr : static_cast<T*>(t->data_ptr());
}

// What every attention call shares: q, k_cache, v_cache, block_table, seq_lens, and the dims.
struct Attention {
  const at::Tensor *q, *k, *v, *table, *lens;
  const at::Tensor* workspace = nullptr;
  size_t workspace_bytes = 0;
  int64_t B, Hq, D;
  bana_dims dims{};

  bool take(Args& a, PyObject* const* o, PyObject* py_dims, long long max_range_tokens) {
    q = a.get(o[0], at::kBFloat16);
    k = a.get(o[1], at::kBFloat16);
    if (q == nullptr || k == nullptr || q->dim() != 3 || k->dim() != 5) return false;
    B = q->size(0), Hq = q->size(1), D = q->size(2);
    const int64_t nb = k->size(0), Hkv = k->size(1), bs = k->size(3);
    if (k->size(2) != D / 8 || k->size(4) != 8) return false;
    v = a.get(o[2], at::kBFloat16, {nb, Hkv, D, bs});
    table = a.get(o[3], at::kInt);
    lens = a.get(o[4], at::kInt, {B});
    if (v == nullptr || table == nullptr || lens == nullptr || table->dim() != 2 || table->size(0) != B) return false;
    bana_dims want{};
    want.batch = (int32_t)B;
    want.num_q_heads = (int32_t)Hq;
    want.num_kv_heads = (int32_t)Hkv;
    want.head_dim = (int32_t)D;
    want.block_size = (int32_t)bs;
    want.max_blocks_per_seq = (int32_t)table->size(1);
    want.num_blocks = nb;
    want.max_range_tokens = (int32_t)max_range_tokens;
    dims = want;
    if (py_dims == Py_None) return true;
    // Caller-built dims must describe the tensors (block_size is the C ABI's to check, as in Python).
    if (Py_TYPE(py_dims) != reinterpret_cast<PyTypeObject*>(g_dims_type)) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(py_dims, &view, PyBUF_SIMPLE) != 0) return false;
    const bool whole = view.len == (Py_ssize_t)sizeof(bana_dims);
    if (whole) dims = *static_cast<const bana_dims*>(view.buf);
    PyBuffer_Release(&view);
    return whole && dims.batch == B && dims.num_q_heads == Hq && dims.num_kv_heads == Hkv && dims.head_dim == D &&
           dims.max_blocks_per_seq == table->size(1) && dims.num_blocks == nb;
  }

  bool take_workspace(Args& a, PyObject* o) {
    if (o == Py_None) return true;
    workspace = a.any(o);
    if (workspace == nullptr) return false;
    workspace_bytes = (size_t)workspace->numel() * workspace->element_size();
    return true;
  }
};

// Runs `call` (status, or -100 for "let Python look") with no exception leaving it.
template <typename F>
PyObject* guarded(F call) {
  long st = -100;
  try {
    st = call();
  } catch (...) {
    st = -100;
  }
  if (st == -100) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  return PyLong_FromLong(st);
}

constexpr long kLook = -100;

#define WITHOUT_GIL(expr)                     \
  [&] {                                       \
    long st_;                                 \
    Py_BEGIN_ALLOW_THREADS st_ = (long)(expr); \
    Py_END_ALLOW_THREADS return st_;          \
  }()

// partial(q, k, v, table, lens, begin, end, out, lse, workspace, stream, dims, max_range_tokens)
PyObject* partial(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    Attention t;
    long long most;
    void* s;
    if (n != 13 || !int_arg(o[12], &most) || !t.take(a, o, o[11], most)) return kLook;
    const at::Tensor *begin = a.get(o[5], at::kInt, {t.B}), *end = a.get(o[6], at::kInt, {t.B});
    const at::Tensor *out = a.get(o[7], at::kFloat, {t.B, t.Hq, t.D}), *lse = a.get(o[8], at::kFloat, {t.B, t.Hq});
    if (!begin || !end || !out || !lse || !t.take_workspace(a, o[9]) || !a.on_current_device() ||
        !stream_handle(o[10], a.device, &s))
      return kLook;
    return WITHOUT_GIL(g_api.partial(&t.dims, data<void>(t.q), data<void>(t.k), data<void>(t.v),
                                     data<int32_t>(t.table), data<int32_t>(t.lens), data<int32_t>(begin),
                                     data<int32_t>(end), data<float>(out), data<float>(lse), data<void>(t.workspace),
                                     t.workspace_bytes, s));
  });
}

// noalloc(q, k, v, table, lens, begin, end, out, lse, stream, dims, max_range_tokens)
PyObject* noalloc(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    Attention t;
    long long most;
    void* s;
    if (n != 12 || !int_arg(o[11], &most) || !t.take(a, o, o[10], most)) return kLook;
    const at::Tensor *begin = a.get(o[5], at::kInt, {t.B}), *end = a.get(o[6], at::kInt, {t.B});
    const at::Tensor *out = a.get(o[7], at::kFloat, {t.B, t.Hq, t.D}), *lse = a.get(o[8], at::kFloat, {t.B, t.Hq});
    if (!begin || !end || !out || !lse || !a.on_current_device() || !stream_handle(o[9], a.device, &s)) return kLook;
    return WITHOUT_GIL(g_api.noalloc(&t.dims, data<void>(t.q), data<void>(t.k), data<void>(t.v),
                                     data<int32_t>(t.table), data<int32_t>(t.lens), data<int32_t>(begin),
                                     data<int32_t>(end), data<float>(out), data<float>(lse), s));
  });
}

// fused(q, k, v, table, lens, begin, end, out, lse, workspace, stream, dims, copies or None)
PyObject* fused(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    Attention t;
    void* s;
    if (n != 13 || !t.take(a, o, o[11], 0)) return kLook;
    const at::Tensor* begin = a.get(o[5], at::kInt);
    if (begin == nullptr || begin->dim() != 2 || begin->size(1) != t.B) return kLook;
    const int64_t parts = begin->size(0);
    const at::Tensor* end = a.get(o[6], at::kInt, {parts, t.B});
    const at::Tensor *out = a.get(o[7], at::kFloat, {t.B, t.Hq, t.D}), *lse = a.get(o[8], at::kFloat, {t.B, t.Hq});
    if (!end || !out || !lse || !t.take_workspace(a, o[9]) || !a.on_current_device() ||
        !stream_handle(o[10], a.device, &s))
      return kLook;
    if (o[12] == Py_None)
      return WITHOUT_GIL(g_api.fused(&t.dims, data<void>(t.q), data<void>(t.k), data<void>(t.v),
                                     data<int32_t>(t.table), data<int32_t>(t.lens), data<int32_t>(begin),
                                     data<int32_t>(end), (int32_t)parts, data<float>(out), data<float>(lse),
                                     data<void>(t.workspace), t.workspace_bytes, s));
    // Copies: pairs (dst, src) of contiguous tensors of one size, each on a device or in pinned memory.
    if (!PyList_CheckExact(o[12]) || PyList_GET_SIZE(o[12]) > kMaxCopies) return kLook;
    const int n_copies = (int)PyList_GET_SIZE(o[12]);
    bana_copy copies[kMaxCopies];
    for (int i = 0; i < n_copies; ++i) {
      PyObject* pair = PyList_GET_ITEM(o[12], i);
      if (!PyTuple_CheckExact(pair) || PyTuple_GET_SIZE(pair) != 2) return kLook;
      const at::Tensor* side[2];
      for (int k = 0; k < 2; ++k) {
        PyObject* x = PyTuple_GET_ITEM(pair, k);
        if (!THPVariable_CheckExact(x)) return kLook;
        side[k] = &THPVariable_Unpack(x);
        if (!side[k]->is_contiguous() || (!side[k]->is_cuda() && !side[k]->is_pinned())) return kLook;
      }
      const size_t bytes = (size_t)side[1]->numel() * side[1]->element_size();
      if ((size_t)side[0]->numel() * side[0]->element_size() != bytes) return kLook;
      copies[i] = bana_copy{side[0]->data_ptr(), side[1]->data_ptr(), bytes};
    }
    return WITHOUT_GIL(g_api.fused_copies(&t.dims, data<void>(t.q), data<void>(t.k), data<void>(t.v),
                                          data<int32_t>(t.table), data<int32_t>(t.lens), data<int32_t>(begin),
                                          data<int32_t>(end), (int32_t)parts, data<float>(out), data<float>(lse),
                                          data<void>(t.workspace), t.workspace_bytes, copies, n_copies, s));
  });
}

// heads(q, k, v, table, lens, begin, end, kv_head_begin, kv_head_end, out, lse, workspace, stream, dims)
PyObject* heads(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    Attention t;
    long long h0, h1;
    void* s;
    if (n != 14 || !int_arg(o[7], &h0) || !int_arg(o[8], &h1) || h0 != (int32_t)h0 || h1 != (int32_t)h1 ||
        !t.take(a, o, o[13], 0))
      return kLook;
    const at::Tensor *begin = a.get(o[5], at::kInt, {t.B}), *end = a.get(o[6], at::kInt, {t.B});
    const at::Tensor *out = a.get(o[9], at::kFloat, {t.B, t.Hq, t.D}), *lse = a.get(o[10], at::kFloat, {t.B, t.Hq});
    if (!begin || !end || !out || !lse || !t.take_workspace(a, o[11]) || !a.on_current_device() ||
        !stream_handle(o[12], a.device, &s))
      return kLook;
    return WITHOUT_GIL(g_api.heads(&t.dims, data<void>(t.q), data<void>(t.k), data<void>(t.v), data<int32_t>(t.table),
                                   data<int32_t>(t.lens), data<int32_t>(begin), data<int32_t>(end), (int32_t)h0,
                                   (int32_t)h1, data<float>(out), data<float>(lse), data<void>(t.workspace),
                                   t.workspace_bytes, s));
  });
}

// merge(out_partials, lses, out, lse_out or None, stream)
PyObject* merge(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    void* s;
    if (n != 5) return kLook;
    const at::Tensor* parts = a.get(o[0], at::kFloat);
    if (parts == nullptr || parts->dim() != 4) return kLook;
    const int64_t P = parts->size(0), B = parts->size(1), Hq = parts->size(2), D = parts->size(3);
    const at::Tensor *lses = a.get(o[1], at::kFloat, {P, B, Hq}), *out = a.get(o[2], at::kFloat, {B, Hq, D});
    const at::Tensor* lse = o[3] == Py_None ? nullptr : a.get(o[3], at::kFloat, {B, Hq});
    if (!lses || !out || (o[3] != Py_None && !lse) || !a.on_current_device() || !stream_handle(o[4], a.device, &s))
      return kLook;
    bana_dims d{};
    d.batch = (int32_t)B;
    d.num_q_heads = (int32_t)Hq;
    d.num_kv_heads = 1;
    d.head_dim = (int32_t)D;
    d.block_size = 16;
    d.max_blocks_per_seq = 1;
    d.num_blocks = 1;
    return WITHOUT_GIL(g_api.merge(&d, data<float>(parts), data<float>(lses), (int32_t)P, data<float>(out),
                                   data<float>(lse), s));
  });
}

// migrate(src_k, src_v, src_table, dst_k, dst_v, dst_table, blk_begin, blk_end, stream, max_range_tokens)
PyObject* migrate(PyObject*, PyObject* const* o, Py_ssize_t n) {
  return guarded([&]() -> long {
    Args a;
    long long most;
    void* s;
    if (n != 10 || !int_arg(o[9], &most)) return kLook;
    constexpr int64_t D = 128;
    const at::Tensor *sk = a.get(o[0], at::kBFloat16), *dk = a.get(o[3], at::kBFloat16);
    if (sk == nullptr || dk == nullptr || sk->dim() != 5 || dk->dim() != 5) return kLook;
    const int64_t nb = sk->size(0), H = sk->size(1), bs = sk->size(3), nbd = dk->size(0);
    if (sk->sizes() != at::IntArrayRef({nb, H, D / 8, bs, 8}) || dk->sizes() != at::IntArrayRef({nbd, H, D / 8, bs, 8}))
      return kLook;
    const at::Tensor *sv = a.get(o[1], at::kBFloat16, {nb, H, D, bs}), *dv = a.get(o[4], at::kBFloat16, {nbd, H, D, bs});
    const at::Tensor* st = a.get(o[2], at::kInt);
    if (!sv || !dv || !st || st->dim() != 2) return kLook;
    const int64_t B = st->size(0), mb = st->size(1);
    const at::Tensor *dt = a.get(o[5], at::kInt, {B, mb}), *jb = a.get(o[6], at::kInt, {B}), *je = a.get(o[7], at::kInt, {B});
    if (!dt || !jb || !je || !a.on_current_device() || !stream_handle(o[8], a.device, &s)) return kLook;
    bana_dims d{};
    d.batch = (int32_t)B;
    d.num_q_heads = d.num_kv_heads = (int32_t)H;
    d.head_dim = (int32_t)D;
    d.block_size = (int32_t)bs;
    d.max_blocks_per_seq = (int32_t)mb;
    d.num_blocks = nb;
    d.max_range_tokens = (int32_t)most;
    return WITHOUT_GIL(g_api.migrate(&d, data<void>(sk), data<void>(sv), data<int32_t>(st), data<void>(dk),
                                     data<void>(dv), data<int32_t>(dt), nbd, data<int32_t>(jb), data<int32_t>(je), s));
  });
}

// setup((address of each C ABI call, in Api's order), raw-stream function, stream type, bana_dims type)
PyObject* setup(PyObject*, PyObject* const* o, Py_ssize_t n) {
  constexpr Py_ssize_t kCalls = sizeof(Api) / sizeof(void*);
  void* address[kCalls];
  if (n != 4 || !PyTuple_CheckExact(o[0]) || PyTuple_GET_SIZE(o[0]) != kCalls) {
    PyErr_SetString(PyExc_TypeError, "setup: a tuple of addresses, the raw-stream function, the stream type and bana_dims");
    return nullptr;
  }
  for (Py_ssize_t i = 0; i < kCalls; ++i) address[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(o[0], i));
  if (PyErr_Occurred()) return nullptr;
  memcpy(&g_api, address, sizeof(g_api));
  Py_INCREF(o[1]);
  Py_XSETREF(g_raw_stream, o[1]);
  Py_INCREF(o[2]);
  Py_XSETREF(g_stream_type, o[2]);
  Py_INCREF(o[3]);
  Py_XSETREF(g_dims_type, o[3]);
  return PyLong_FromSize_t(sizeof(bana_dims));
}

#define METHOD(f) {#f, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL, nullptr}
PyMethodDef g_methods[] = {METHOD(setup), METHOD(partial), METHOD(noalloc), METHOD(fused), METHOD(heads),
                           METHOD(merge), METHOD(migrate), {nullptr, nullptr, 0, nullptr}};
PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_native", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__native(void) { return PyModule_Create(&g_module); }
