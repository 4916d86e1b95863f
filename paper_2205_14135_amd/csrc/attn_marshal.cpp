// Argument marshalling of the binding's forward and backward calls (paper_2205_14135_amd/binding.py)
// as a CPython extension: tensor checks, output allocation, parameter block and the library call in
// one native call.  The same steps in Python and ctypes took 9 us of a forward call with its
// buffers given, and 30 + 46 us of a training step through autograd, whose backward runs on the engine's own
// thread with cold caches; a small problem's kernels take 5 to 10 us each.  A pass with the one binding and with the other, over
// the same library, in turn: one forward call of one head of 128 tokens 9.5 -> 4.6 us, a training step of 96 heads of 197 tokens
// 149 -> 85 us (4 % between runs), of a padded batch of 128 heads of up to 700 tokens 147 -> 86 us (6 %).
// The autograd node of flash_attention (paper_2205_14135_amd/autograd.py) is here too: the engine runs backwards on a thread
// of its own, and a node in Python waits there for the interpreter lock, twice, with cold caches.  Host time of a training step of 96
// heads of 197 tokens, node in Python | here: 82 | 64 us, or 39 | 34 where the machine happens to run both threads close together (33 us
// and more of either are the engine's own change of threads: so much takes the backward of a single product).
// The functions take positional arguments only (binding.py holds the public signatures and
// defaults) and raise what the Python marshalling of the measurement entry points raises: ValueError, TypeError, AttnError.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/custom_function.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <initializer_list>

#include "../../include/attn.h"

namespace {

// Entry points of the library that binding.load() opened.
struct Library {
  decltype(&attn_fwd) fwd = nullptr;
  decltype(&attn_bwd) bwd = nullptr;
  decltype(&attn_bwd_workspace_bytes) workspace_bytes = nullptr;
  decltype(&attn_blocksparse_fwd) sparse_fwd = nullptr;
  decltype(&attn_blocksparse_bwd) sparse_bwd = nullptr;
  decltype(&attn_blocksparse_bwd_workspace_bytes) sparse_workspace_bytes = nullptr;
};
Library lib;
PyObject* attn_error = nullptr;   // binding.AttnError

struct Raised {};   // a Python error is set

[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw Raised();
}

void check_status(int status, const char* where) {
  if (status == ATTN_OK) return;
  PyObject* e = PyObject_CallFunction(attn_error, "is", status, where);
  if (e != nullptr) {
    PyErr_SetObject(attn_error, e);
    Py_DECREF(e);
  }
  throw Raised();
}

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a torch.Tensor");
  return THPVariable_Unpack(o);
}
void* data(PyObject* o) {   // of a buffer the library checks for: None is its NULL
  return o == Py_None ? nullptr : tensor(o).data_ptr();
}
PyObject* wrap(const at::Tensor& t) {
  PyObject* o = THPVariable_Wrap(t);
  if (o == nullptr) throw Raised();
  return o;
}
double number(PyObject* o) {   // float(o)
  PyObject* f = PyNumber_Float(o);
  if (f == nullptr) throw Raised();
  const double v = PyFloat_AS_DOUBLE(f);
  Py_DECREF(f);
  return v;
}
bool truth(PyObject* o) {
  const int v = PyObject_IsTrue(o);
  if (v < 0) throw Raised();
  return v != 0;
}
uint64_t low64(PyObject* o) {   // int(o) & (2^64 - 1)
  PyObject* i = PyNumber_Long(o);
  if (i == nullptr) throw Raised();
  const uint64_t v = PyLong_AsUnsignedLongLongMask(i);
  Py_DECREF(i);
  if (v == (uint64_t)-1 && PyErr_Occurred()) throw Raised();
  return v;
}

bool alike(const at::Tensor& ref, const at::Tensor& t) {
  return t.sizes() == ref.sizes() && t.strides() == ref.strides() && t.device() == ref.device();
}
void same_layout(const at::Tensor& ref, const at::Tensor& t) {
  if (!alike(ref, t)) raise(PyExc_ValueError, "all [B,H,N,d] tensors must share shape, strides and device");
}

// The arguments that every call has, in the order of the Python wrappers.
struct Options {
  PyObject *softmax_scale, *causal, *dropout_p, *seed, *offset, *o_fp32, *stream, *key_lengths;
};
Options options(PyObject* const* a) { return {a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7]}; }
constexpr Py_ssize_t kOptions = 8;

attn_params make_params(PyObject* q_object, const Options& o) {
  const at::Tensor& q = tensor(q_object);
  if (q.dim() != 4 || q.stride(3) != 1) raise(PyExc_ValueError, "expected a [B,H,N,d] tensor with contiguous last axis");
  attn_params p = {};
  p.B = (int32_t)q.size(0); p.H = (int32_t)q.size(1); p.N = (int32_t)q.size(2); p.d = (int32_t)q.size(3);
  if (q.scalar_type() == at::kHalf) p.dtype = ATTN_FP16;
  else if (q.scalar_type() == at::kBFloat16) p.dtype = ATTN_BF16;
  else {
    PyObject* dtype = PyObject_GetAttrString(q_object, "dtype");
    if (dtype == nullptr) throw Raised();
    PyErr_Format(PyExc_TypeError, "Q/K/V must be float16 or bfloat16, got %S", dtype);
    Py_DECREF(dtype);
    throw Raised();
  }
  p.stride_b = q.stride(0); p.stride_h = q.stride(1); p.stride_n = q.stride(2);
  p.softmax_scale = (float)number(o.softmax_scale);
  p.causal = truth(o.causal);
  p.dropout_p = (float)number(o.dropout_p);
  p.seed = low64(o.seed);
  p.offset = low64(o.offset);
  p.o_fp32 = truth(o.o_fp32);
  if (o.stream != Py_None) p.stream = (void*)(uintptr_t)low64(o.stream);
  else if (q.is_cuda()) p.stream = (void*)c10::hip::getCurrentHIPStream(q.device().index()).stream();
  if (o.key_lengths != Py_None) {
    const at::Tensor& k = tensor(o.key_lengths);
    if (k.scalar_type() != at::kInt || k.dim() != 1 || k.size(0) != q.size(0) || !k.is_contiguous())
      raise(PyExc_TypeError, "key_lengths must be a contiguous int32 tensor of shape [B]");
    p.key_lengths = (const int32_t*)k.data_ptr();
  }
  return p;
}

// Block mask arguments of the block-sparse calls: mask tensor, mask_block.
struct Mask { const uint8_t* ptr; int32_t block; int64_t stride_h; };
Mask mask_args(PyObject* mask, PyObject* mask_block, int64_t H) {
  const at::Tensor& m = tensor(mask);
  if (m.scalar_type() != at::kByte || !m.is_contiguous())
    raise(PyExc_TypeError, "block_mask must be a contiguous uint8 tensor [T,T] or [H,T,T]");
  Mask r = {nullptr, (int32_t)low64(mask_block), 0};
  if (m.dim() == 3 && m.size(0) == H) r.stride_h = m.stride(0);
  else if (m.dim() != 2) raise(PyExc_ValueError, "block_mask must be [T,T] or [H,T,T]");
  r.ptr = (const uint8_t*)m.data_ptr();
  return r;
}

at::Tensor like(const at::Tensor& q, at::ScalarType type) {
  return at::empty_strided(q.sizes(), q.strides(), q.options().dtype(type));
}

// The library call itself runs without the interpreter lock.
template <typename F> int without_gil(F&& f) {
  PyThreadState* s = PyEval_SaveThread();
  const int status = f();
  PyEval_RestoreThread(s);
  return status;
}

void expect_args(Py_ssize_t n, Py_ssize_t want) {
  if (n != want || lib.fwd == nullptr) raise(PyExc_TypeError, "internal call with the wrong arguments, or before attach()");
}

template <typename F> PyObject* guarded(F&& f) {
  HANDLE_TH_ERRORS
  try {
    return f();
  } catch (const Raised&) {
    return nullptr;
  }
  END_HANDLE_TH_ERRORS
}

PyObject* tuple(std::initializer_list<PyObject*> items) {   // takes the references over
  PyObject* t = PyTuple_New((Py_ssize_t)items.size());
  if (t == nullptr) throw Raised();
  Py_ssize_t i = 0;
  for (PyObject* o : items) PyTuple_SET_ITEM(t, i++, o);
  return t;
}

// ---- autograd: the forward call keeps what the backward one needs (the O(N) state: O, the row statistic and the generator state)

// What a backward call takes from its forward call beside the saved tensors.
struct Attention {
  attn_params p;            // pointers (stream, key lengths) are set again for each call
  at::Tensor key_lengths, block_mask;
};

attn_params on_current_stream(const Attention& a, const at::Tensor& q) {
  attn_params p = a.p;
  p.stride_b = q.stride(0); p.stride_h = q.stride(1); p.stride_n = q.stride(2);
  p.stream = (void*)c10::hip::getCurrentHIPStream(q.device().index()).stream();
  p.key_lengths = a.key_lengths.defined() ? (const int32_t*)a.key_lengths.data_ptr() : nullptr;
  return p;
}
int64_t mask_stride(const at::Tensor& mask) { return mask.dim() == 3 ? mask.stride(0) : 0; }

// An error on the engine's thread, which runs without the interpreter lock: `set` raises it, and it is carried to the caller of backward().
template <typename F> [[noreturn]] void refused_in_backward(F&& set) {
  const PyGILState_STATE gil = PyGILState_Ensure();
  python_error e;
  try {
    set();
  } catch (const Raised&) {
    e.persist();
  }
  PyGILState_Release(gil);
  throw e;
}

// What the marshalling of a backward call asks of its tensors (backward() below, make_params), of the saved ones as they come back: hooks
// of the program may have moved, converted or laid out anew some of them, or have given them another batch than the lengths and the masks are for.
void check_saved(const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const at::Tensor& d_out, const Attention& a) {
  if (q.dim() != 4 || q.stride(3) != 1)
    refused_in_backward([] { raise(PyExc_ValueError, "expected a [B,H,N,d] tensor with contiguous last axis"); });
  if (q.scalar_type() != at::kHalf && q.scalar_type() != at::kBFloat16)
    refused_in_backward([] { raise(PyExc_TypeError, "Q/K/V must be float16 or bfloat16"); });
  if (!q.is_cuda()) refused_in_backward([] { raise(PyExc_ValueError, "the saved tensors are not on the GPU"); });
  if (!alike(q, k) || !alike(q, v) || !alike(q, d_out))
    refused_in_backward([] { raise(PyExc_ValueError, "all [B,H,N,d] tensors must share shape, strides and device"); });
  if (a.key_lengths.defined() && a.key_lengths.size(0) != q.size(0))
    refused_in_backward([] { raise(PyExc_TypeError, "key_lengths must be a contiguous int32 tensor of shape [B]"); });
  if (a.block_mask.defined() && a.block_mask.dim() == 3 && a.block_mask.size(0) != q.size(1))
    refused_in_backward([] { raise(PyExc_ValueError, "block_mask must be [T,T] or [H,T,T]"); });
}

using torch::autograd::AutogradContext;
using torch::autograd::variable_list;

struct FlashAttention : torch::autograd::Function<FlashAttention> {
  static at::Tensor forward(AutogradContext* ctx, const at::Tensor& q, const at::Tensor& k, const at::Tensor& v, const Attention& a) {
    const bool sparse = a.block_mask.defined();
    const attn_params p = on_current_stream(a, q);
    const at::Tensor out = like(q, q.scalar_type()), lse = at::empty(q.sizes().slice(0, 3), q.options().dtype(at::kFloat));
    const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
    void* op = out.data_ptr();
    float* lp = (float*)lse.data_ptr();
    check_status(without_gil([&] {
      return sparse ? lib.sparse_fwd(&p, (const uint8_t*)a.block_mask.data_ptr(), 128, mask_stride(a.block_mask), qp, kp, vp, op, lp)
                    : lib.fwd(&p, qp, kp, vp, op, lp);
    }), sparse ? "attn_blocksparse_fwd" : "attn_fwd");
    ctx->save_for_backward({q, k, v, out, lse});
    auto& data = ctx->saved_data;
    data["softmax_scale"] = (double)a.p.softmax_scale;
    data["causal"] = a.p.causal != 0;
    data["dropout_p"] = (double)a.p.dropout_p;
    data["seed"] = (int64_t)a.p.seed;
    data["offset"] = (int64_t)a.p.offset;
    if (a.key_lengths.defined()) data["key_lengths"] = a.key_lengths;
    if (sparse) data["block_mask"] = a.block_mask;
    return out;
  }

  static variable_list backward(AutogradContext* ctx, const variable_list& d_outs) {
    const variable_list saved = ctx->get_saved_variables();
    const at::Tensor &q = saved[0], &k = saved[1], &v = saved[2], &out = saved[3], &lse = saved[4];
    at::Tensor d_out = d_outs[0];
    if (d_out.sizes() != q.sizes() || d_out.strides() != q.strides())   // the library addresses dO with the strides of q
      d_out = like(q, q.scalar_type()).copy_(d_out);
    auto& data = ctx->saved_data;
    Attention a = {};
    if (data.count("key_lengths")) a.key_lengths = data["key_lengths"].toTensor();
    if (data.count("block_mask")) a.block_mask = data["block_mask"].toTensor();
    check_saved(q, k, v, d_out, a);
    a.p.B = (int32_t)q.size(0); a.p.H = (int32_t)q.size(1); a.p.N = (int32_t)q.size(2); a.p.d = (int32_t)q.size(3);
    a.p.dtype = q.scalar_type() == at::kHalf ? ATTN_FP16 : ATTN_BF16;
    a.p.softmax_scale = (float)data["softmax_scale"].toDouble();
    a.p.causal = data["causal"].toBool();
    a.p.dropout_p = (float)data["dropout_p"].toDouble();
    a.p.seed = (uint64_t)data["seed"].toInt();
    a.p.offset = (uint64_t)data["offset"].toInt();
    const bool sparse = a.block_mask.defined();
    const attn_params p = on_current_stream(a, q);
    at::Tensor g[3];
    for (at::Tensor& t : g) t = like(q, q.scalar_type());
    const size_t need = sparse ? lib.sparse_workspace_bytes(&p) : lib.workspace_bytes(&p);
    const at::Tensor ws = at::empty({(int64_t)std::max<size_t>(need, 256)}, q.options().dtype(at::kByte));
    const float* lp = (const float*)lse.data_ptr();
    const int status =
        sparse ? lib.sparse_bwd(&p, (const uint8_t*)a.block_mask.data_ptr(), 128, mask_stride(a.block_mask), q.data_ptr(), k.data_ptr(), v.data_ptr(),
                                out.data_ptr(), d_out.data_ptr(), lp, g[0].data_ptr(), g[1].data_ptr(), g[2].data_ptr(), ws.data_ptr(), ws.numel())
               : lib.bwd(&p, q.data_ptr(), k.data_ptr(), v.data_ptr(), out.data_ptr(), d_out.data_ptr(), lp, g[0].data_ptr(), g[1].data_ptr(),
                         g[2].data_ptr(), ws.data_ptr(), ws.numel());
    if (status != ATTN_OK) refused_in_backward([&] { check_status(status, sparse ? "attn_blocksparse_bwd" : "attn_bwd"); });
    return {g[0], g[1], g[2], at::Tensor()};
  }
};

// attention(Q, K, V, softmax_scale, causal, dropout_p, seed, offset, key_lengths, block_mask) -> O, differentiable
PyObject* py_attention(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 10);
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    same_layout(q, k);
    same_layout(q, v);
    Attention at = {};
    at.p = make_params(a[0], {a[3], a[4], a[5], a[6], a[7], Py_False, Py_None, a[8]});
    if (a[8] != Py_None) at.key_lengths = tensor(a[8]);
    if (a[9] != Py_None) {
      PyObject* block = PyLong_FromLong(128);
      if (block == nullptr) throw Raised();
      try {
        mask_args(a[9], block, q.size(1));
      } catch (...) {
        Py_DECREF(block);
        throw;
      }
      Py_DECREF(block);
      at.block_mask = tensor(a[9]);
    }
    return wrap(FlashAttention::apply(q, k, v, at));
  });
}

// fwd(Q, K, V, <options>, out, lse[, block_mask, mask_block]) -> (O, LSE)
PyObject* forward(PyObject* const* a, Py_ssize_t n, bool sparse) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 3 + kOptions + 2 + (sparse ? 2 : 0));
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]);
    same_layout(q, k);
    same_layout(q, v);
    const attn_params p = make_params(a[0], options(a + 3));
    PyObject* const* r = a + 3 + kOptions;
    Mask m = {};
    if (sparse) m = mask_args(r[2], r[3], q.size(1));
    const at::Tensor out = r[0] != Py_None ? tensor(r[0]) : like(q, p.o_fp32 ? at::kFloat : q.scalar_type());
    const at::Tensor lse = r[1] != Py_None ? tensor(r[1]) : at::empty(q.sizes().slice(0, 3), q.options().dtype(at::kFloat));
    const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr();
    void* op = out.data_ptr();
    float* lp = (float*)lse.data_ptr();
    check_status(without_gil([&] {
      return sparse ? lib.sparse_fwd(&p, m.ptr, m.block, m.stride_h, qp, kp, vp, op, lp) : lib.fwd(&p, qp, kp, vp, op, lp);
    }), sparse ? "attn_blocksparse_fwd" : "attn_fwd");
    return tuple({r[0] != Py_None ? Py_NewRef(r[0]) : wrap(out), r[1] != Py_None ? Py_NewRef(r[1]) : wrap(lse)});
  });
}

// bwd(Q, K, V, O, dO, LSE, <options>, workspace, allocate, dQ, dK, dV[, block_mask, mask_block]) -> (dQ, dK, dV);
// allocate: dQ, dK and dV are made here, else they are the caller's
PyObject* backward(PyObject* const* a, Py_ssize_t n, bool sparse) {
  return guarded([&]() -> PyObject* {
    expect_args(n, 6 + kOptions + 5 + (sparse ? 2 : 0));
    const at::Tensor &q = tensor(a[0]), &k = tensor(a[1]), &v = tensor(a[2]), &go = tensor(a[4]);
    same_layout(q, k);
    same_layout(q, v);
    same_layout(q, go);
    const attn_params p = make_params(a[0], options(a + 6));
    PyObject* const* r = a + 6 + kOptions;
    Mask m = {};
    if (sparse) m = mask_args(r[5], r[6], q.size(1));
    const bool allocate = truth(r[1]);
    at::Tensor g[3];
    void* gp[3];
    for (int i = 0; i < 3; ++i) {
      if (allocate) g[i] = like(q, q.scalar_type());
      gp[i] = allocate ? g[i].data_ptr() : data(r[2 + i]);
    }
    at::Tensor ws;
    if (r[0] != Py_None) {
      ws = tensor(r[0]);
    } else {
      const size_t need = sparse ? lib.sparse_workspace_bytes(&p) : lib.workspace_bytes(&p);
      ws = at::empty({(int64_t)std::max<size_t>(need, 256)}, q.options().dtype(at::kByte));
    }
    const size_t ws_bytes = (size_t)ws.numel() * ws.element_size();
    const void *qp = q.data_ptr(), *kp = k.data_ptr(), *vp = v.data_ptr(), *op = data(a[3]), *gop = go.data_ptr();
    const float* lp = (const float*)data(a[5]);
    void* wp = ws.data_ptr();
    check_status(without_gil([&] {
      return sparse ? lib.sparse_bwd(&p, m.ptr, m.block, m.stride_h, qp, kp, vp, op, gop, lp, gp[0], gp[1], gp[2], wp, ws_bytes)
                    : lib.bwd(&p, qp, kp, vp, op, gop, lp, gp[0], gp[1], gp[2], wp, ws_bytes);
    }), sparse ? "attn_blocksparse_bwd" : "attn_bwd");
    PyObject* t[3];
    for (int i = 0; i < 3; ++i) t[i] = allocate ? wrap(g[i]) : Py_NewRef(r[2 + i]);
    return tuple({t[0], t[1], t[2]});
  });
}

PyObject* py_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) { return forward(a, n, false); }
PyObject* py_sparse_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) { return forward(a, n, true); }
PyObject* py_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) { return backward(a, n, false); }
PyObject* py_sparse_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) { return backward(a, n, true); }

// attach(AttnError, address of attn_fwd, attn_bwd, attn_bwd_workspace_bytes, and the three block-sparse ones)
PyObject* py_attach(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded([&]() -> PyObject* {
    if (n != 7) raise(PyExc_TypeError, "attach() takes the error class and six addresses");
    Library l;
    l.fwd = (decltype(l.fwd))low64(a[1]);
    l.bwd = (decltype(l.bwd))low64(a[2]);
    l.workspace_bytes = (decltype(l.workspace_bytes))low64(a[3]);
    l.sparse_fwd = (decltype(l.sparse_fwd))low64(a[4]);
    l.sparse_bwd = (decltype(l.sparse_bwd))low64(a[5]);
    l.sparse_workspace_bytes = (decltype(l.sparse_workspace_bytes))low64(a[6]);
    Py_INCREF(a[0]);
    Py_XDECREF(attn_error);
    attn_error = a[0];
    lib = l;
    Py_RETURN_NONE;
  });
}

PyMethodDef methods[] = {
    {"attach", (PyCFunction)(void*)py_attach, METH_FASTCALL, nullptr},
    {"attention", (PyCFunction)(void*)py_attention, METH_FASTCALL, nullptr},
    {"fwd", (PyCFunction)(void*)py_fwd, METH_FASTCALL, nullptr},
    {"bwd", (PyCFunction)(void*)py_bwd, METH_FASTCALL, nullptr},
    {"blocksparse_fwd", (PyCFunction)(void*)py_sparse_fwd, METH_FASTCALL, nullptr},
    {"blocksparse_bwd", (PyCFunction)(void*)py_sparse_bwd, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal(void) { return PyModule_Create(&module); }
