// The Python face's native half: takes a call's arguments apart (torch tensors, NumPy arrays, ba_heads) and makes
// the call.  Each function takes exactly what the Python function of its name takes and returns the call's status,
// or None where an argument is anything but the plain case (a tensor subclass, a list for an array, a shape that
// does not fit the call): nothing has been launched then, and the Python function goes through its own checks,
// which convert what can be converted and say what is wrong with the rest.
//
// A call of a few microseconds on the device spent more on this in Python: 5 us of 12 for per-block encoding, 6 of 15
// for a final block, 19 of 39 for encoding, re-encoding and final block of one prompt.
//
// It sees inside torch's tensors, so it serves the torch it was built with and no other: torch_version.
#define NPY_NO_DEPRECATED_API NPY_1_7_API_VERSION
#include <Python.h>

#include <numpy/arrayobject.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/version.h>

#include <cxxabi.h>

#include <algorithm>
#include <cstring>
#include <new>
#include <vector>

#include "../../include/ba.h"

namespace {

// The library's entry points (loaded by the Python face, which hands over their addresses).
struct {
  decltype(&ba_encode_blocks) encode;
  decltype(&ba_reencode_positions) reencode;
  decltype(&ba_final_block_attention) final_block;
  decltype(&ba_final_block_attention_static) final_static;
  decltype(&ba_final_block_attention_cached) final_cached;
  decltype(&ba_block_attention_prompts) prompts;
  decltype(&ba_block_attention_prompts_backward) prompts_backward;
} lib;
PyTypeObject *heads_type;
PyObject *name_c, *name_cuda_stream, *get_device, *get_raw_stream;

// Arguments that are not the plain case.
struct Declined {};
void need(bool ok) {
  if (!ok) throw Declined();
}

// The ba_heads inside a Heads object, held for the call.
struct HeadsArg {
  Py_buffer view{};
  const ba_heads *h = nullptr;
  explicit HeadsArg(PyObject *o) {
    need(Py_TYPE(o) == heads_type);
    PyObject *c = PyObject_GetAttr(o, name_c);
    need(c != nullptr);
    const int rc = PyObject_GetBuffer(c, &view, PyBUF_SIMPLE);  // (the view holds a reference of its own)
    Py_DECREF(c);
    need(rc == 0);
    if (view.len != (Py_ssize_t)sizeof(ba_heads)) {
      PyBuffer_Release(&view);
      throw Declined();
    }
    h = (const ba_heads *)view.buf;
  }
  ~HeadsArg() { PyBuffer_Release(&view); }
  HeadsArg(const HeadsArg &) = delete;
};

bool is_int32_array(PyObject *o) {
  if (!PyArray_CheckExact(o)) return false;
  PyArrayObject *a = (PyArrayObject *)o;
  return PyArray_TYPE(a) == NPY_INT32 && PyArray_NDIM(a) == 1 && PyArray_ISCARRAY_RO(a);
}
// int32 host array (as guarded has seen) or None, copied: the call runs without the interpreter's lock.
struct Ints {
  int32_t few[96];
  std::vector<int32_t> many;
  const int32_t *p = nullptr;
  int64_t n = 0;
  explicit Ints(PyObject *o) {
    if (o == Py_None) return;
    PyArrayObject *a = (PyArrayObject *)o;
    n = PyArray_DIM(a, 0);
    const int32_t *from = (const int32_t *)PyArray_DATA(a);
    int32_t *to = few;
    if (n > (int64_t)(sizeof(few) / 4)) {
      many.resize((size_t)n);
      to = many.data();
    }
    if (n) memcpy(to, from, (size_t)n * 4);
    p = to;
  }
  Ints(const Ints &) = delete;
  int64_t last() const { return n ? p[n - 1] : 0; }
};
void same_len(int64_t n, const Ints &a) { need(!a.p || a.n == n); }
// rows that blocks [off, off + len) reach (empty blocks touch nothing)
int64_t reach(const Ints &off, const Ints &len) {
  if (!off.p || !len.p || !len.n) return 0;
  need(off.n == len.n);
  int64_t most = 0;
  bool any = false;
  for (int64_t i = 0; i < len.n; ++i)
    if (len.p[i] > 0) {
      const int64_t end = (int64_t)off.p[i] + len.p[i];
      most = any ? std::max(most, end) : end;
      any = true;
    }
  return most;
}

const at::Tensor &plain_tensor(PyObject *o) {
  need(THPVariable_CheckExact(o));
  const at::Tensor &t = THPVariable_Unpack(o);
  need(t.defined() && t.is_cuda() && t.layout() == at::kStrided);
  return t;
}
// [tokens, heads, D] on the GPU, D contiguous, with the call's heads and at least the rows it reaches; with `layers`
// the first layer of a [layers, tokens, heads, D] one.
struct TensorArg {
  ba_tensor t{};
  const ba_tensor *p = nullptr;
  TensorArg(PyObject *o, int64_t heads, int64_t d, int64_t min_tokens, bool allow_f32 = false, bool layers = false) {
    if (o == Py_None) return;
    const at::Tensor &x = plain_tensor(o);
    const auto type = x.scalar_type();
    need(type == at::kBFloat16 || (allow_f32 && type == at::kFloat));
    const auto size = x.sizes(), stride = x.strides();
    const size_t at = layers ? 1 : 0;
    need(size.size() == at + 3);
    need(size[at + 2] <= 1 || stride[at + 2] == 1);
    need(size[at + 1] == heads && size[at + 2] == d && size[at] >= min_tokens);
    t.ptr = x.data_ptr();
    t.stride_tok = stride[at];
    t.stride_head = stride[at + 1];
    t.dtype = type == at::kFloat ? BA_DTYPE_F32 : BA_DTYPE_BF16;
    p = &t;
  }
  TensorArg(const TensorArg &) = delete;
};
float *lse_of(PyObject *o, int64_t tokens, int64_t n_q_heads) {
  if (o == Py_None) return nullptr;
  const at::Tensor &x = plain_tensor(o);
  need(x.scalar_type() == at::kFloat && x.dim() == 2 && x.is_contiguous() && x.size(1) == n_q_heads && x.size(0) >= tokens);
  return (float *)x.data_ptr();
}
struct Workspace {
  void *p = nullptr;
  size_t bytes = 0;
  explicit Workspace(PyObject *o) {
    if (o == Py_None) return;
    const at::Tensor &x = plain_tensor(o);
    need(x.is_contiguous());
    p = x.data_ptr();
    bytes = (size_t)x.numel() * x.element_size();
  }
};
int32_t int_of(PyObject *o) {
  need(PyLong_CheckExact(o));
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(o, &overflow);
  need(!overflow && v == (int32_t)v);
  return (int32_t)v;
}
void *stream_of(PyObject *o) {
  PyObject *h = nullptr;
  if (o != Py_None) {
    h = PyObject_GetAttr(o, name_cuda_stream);
  } else {
    need(get_raw_stream != nullptr);
    PyObject *dev = PyObject_CallNoArgs(get_device);
    need(dev != nullptr);
    h = PyObject_CallOneArg(get_raw_stream, dev);
    Py_DECREF(dev);
  }
  need(h != nullptr);
  void *s = PyLong_Check(h) ? PyLong_AsVoidPtr(h) : nullptr;
  const bool ok = PyLong_Check(h) && !PyErr_Occurred();
  Py_DECREF(h);
  need(ok);
  return s;
}

// An exception out of the library: its call may have launched something, so it is an error and never "not the plain case".
struct Threw {
  bool memory;
};
// body() makes the call and returns its status.  Arguments 1 .. tensors are tensors or None, those from there to `arrays`
// int32 arrays or None: looked at first, without an exception, which costs 3.5 us (lists and 64-bit arrays are ordinary arguments).
template <typename Body>
PyObject *guarded(PyObject *const *a, Py_ssize_t n, Py_ssize_t want, int tensors, int arrays, Body &&body) {
  if (n != want) Py_RETURN_NONE;
  for (int i = 1; i <= arrays; ++i)
    if (a[i] != Py_None && !(i <= tensors ? THPVariable_CheckExact(a[i]) : is_int32_array(a[i]))) Py_RETURN_NONE;
  try {
    return PyLong_FromLong(body());
  } catch (const Threw &t) {
    PyErr_SetString(t.memory ? PyExc_MemoryError : PyExc_RuntimeError, "an exception inside the library");
    return nullptr;
  } catch (abi::__forced_unwind &) {  // (a thread that ends with the interpreter, waiting for its lock)
    throw;
  } catch (...) {
    PyErr_Clear();  // (the Python function meets the same argument again and raises what there is to raise)
  }
  Py_RETURN_NONE;
}
template <typename Call>
int32_t unlocked(Call &&call) {
  int32_t rc = 0;
  int threw = 0;
  PyThreadState *const state = PyEval_SaveThread();
  try {
    rc = call();
  } catch (const std::bad_alloc &) {
    threw = 2;
  } catch (...) {
    threw = 1;
  }
  PyEval_RestoreThread(state);
  if (threw) throw Threw{threw == 2};
  return rc;
}

PyObject *encode_blocks(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 10, 5, 6, [&] {
    const HeadsArg h(a[0]);
    const Ints offs(a[6]);
    need(offs.p && offs.n > 0);
    const int64_t T = offs.last(), hq = h.h->n_q_heads, hkv = h.h->n_kv_heads, d = h.h->head_dim;
    const TensorArg q(a[1], hq, d, T), k(a[2], hkv, d, T), v(a[3], hkv, d, T), o(a[4], hq, d, T), kl(a[5], hkv, d, T);
    const int32_t mode = int_of(a[7]);
    const Workspace ws(a[8]);
    void *const stream = stream_of(a[9]);
    return unlocked([&] {
      return lib.encode(h.h, q.p, k.p, v.p, o.p, kl.p, (int32_t)(offs.n - 1), offs.p, mode, ws.p, ws.bytes, stream);
    });
  });
}

PyObject *reencode_positions(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 10, 2, 7, [&] {
    const HeadsArg h(a[0]);
    const at::Tensor &s = plain_tensor(a[1]), &t = plain_tensor(a[2]);
    const bool layers = s.dim() == 4;
    need(s.dim() == t.dim() && (layers ? s.size(0) == t.size(0) && s.size(0) > 0 : s.dim() == 3));
    const Ints so(a[3]), to(a[4]), ln(a[5]), op(a[6]), np(a[7]);
    need(so.p && to.p && ln.p);
    for (const Ints *x : {&so, &to, &op, &np}) same_len(ln.n, *x);
    const int64_t hkv = h.h->n_kv_heads, d = h.h->head_dim;
    const TensorArg src(a[1], hkv, d, reach(so, ln), true, layers), dst(a[2], hkv, d, reach(to, ln), true, layers);
    // (one layer: the stride that a view with a leading dimension of one has)
    const int64_t n_layers = layers ? s.size(0) : 1;
    need(n_layers <= INT32_MAX && ln.n <= INT32_MAX);
    const int64_t sl = layers ? s.stride(0) : s.size(0) * s.stride(0), tl = layers ? t.stride(0) : t.size(0) * t.stride(0);
    const int32_t mode = int_of(a[8]);
    void *const stream = stream_of(a[9]);
    return unlocked([&] {
      return lib.reencode(h.h, src.p, dst.p, (int32_t)n_layers, sl, tl, (int32_t)ln.n, so.p, to.p, ln.p, op.p, np.p, mode, stream);
    });
  });
}

// ba_final_block_attention and, without a workspace, ba_final_block_attention_static
template <bool kStatic>
PyObject *final_block(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, kStatic ? 13 : 14, 7, 10, [&] {
    const HeadsArg h(a[0]);
    const Ints cq(a[8]), cc(a[9]), qp(a[10]);
    need(cq.p && cc.p && cq.n > 0 && cq.n == cc.n);
    same_len(cq.n - 1, qp);
    const int64_t hq = h.h->n_q_heads, hkv = h.h->n_kv_heads, d = h.h->head_dim, tq = cq.last(), tc = cc.last();
    const TensorArg q(a[1], hq, d, tq), kc(a[2], hkv, d, tc), vc(a[3], hkv, d, tc), kf(a[4], hkv, d, tq), vf(a[5], hkv, d, tq),
        o(a[6], hq, d, tq), kr(a[7], hkv, d, tq);
    const int32_t mode = int_of(a[11]);
    const Workspace ws(kStatic ? Py_None : a[12]);
    void *const stream = stream_of(a[kStatic ? 12 : 13]);
    return unlocked([&] {
      const int32_t np = (int32_t)(cq.n - 1);
      return kStatic ? lib.final_static(h.h, q.p, kc.p, vc.p, kf.p, vf.p, o.p, kr.p, np, cq.p, cc.p, qp.p, mode, stream)
                     : lib.final_block(h.h, q.p, kc.p, vc.p, kf.p, vf.p, o.p, kr.p, np, cq.p, cc.p, qp.p, mode, ws.p, ws.bytes, stream);
    });
  });
}

PyObject *final_block_cached(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 18, 7, 14, [&] {
    const HeadsArg h(a[0]);
    const Ints cq(a[8]), cb(a[9]), bo(a[10]), bl(a[11]), op(a[12]), np(a[13]), qp(a[14]);
    need(cq.p && cb.p && bo.p && bl.p && cq.n > 0 && cq.n == cb.n);
    for (const Ints *x : {&bo, &bl, &op, &np}) same_len(cb.last(), *x);
    same_len(cq.n - 1, qp);
    const int64_t hq = h.h->n_q_heads, hkv = h.h->n_kv_heads, d = h.h->head_dim, tq = cq.last(), tc = reach(bo, bl);
    const TensorArg q(a[1], hq, d, tq), kc(a[2], hkv, d, tc), vc(a[3], hkv, d, tc), kf(a[4], hkv, d, tq), vf(a[5], hkv, d, tq),
        o(a[6], hq, d, tq), kr(a[7], hkv, d, tq);
    const Workspace ws(a[15]);
    void *const stream = stream_of(a[16]);
    const int32_t below = int_of(a[17]);
    return unlocked([&] {
      return lib.final_cached(h.h, q.p, kc.p, vc.p, kf.p, vf.p, o.p, kr.p, (int32_t)(cq.n - 1), cq.p, cb.p, bo.p, bl.p, op.p, np.p, qp.p,
                              below, ws.p, ws.bytes, stream);
    });
  });
}

PyObject *prompts(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 12, 6, 8, [&] {
    const HeadsArg h(a[0]);
    const Ints cb(a[7]), offs(a[8]);
    need(cb.p && offs.p && cb.n > 0 && offs.n > 0 && cb.last() == offs.n - 1);
    const int64_t T = offs.last(), hq = h.h->n_q_heads, hkv = h.h->n_kv_heads, d = h.h->head_dim;
    const TensorArg q(a[1], hq, d, T), k(a[2], hkv, d, T), v(a[3], hkv, d, T), o(a[4], hq, d, T), kr(a[5], hkv, d, T);
    float *const lse = lse_of(a[6], T, hq);
    const int32_t mode = int_of(a[9]);
    const Workspace ws(a[10]);
    void *const stream = stream_of(a[11]);
    return unlocked([&] {
      return lib.prompts(h.h, q.p, k.p, v.p, o.p, kr.p, lse, (int32_t)(cb.n - 1), cb.p, offs.p, mode, ws.p, ws.bytes, stream);
    });
  });
}

PyObject *prompts_backward(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return guarded(a, n, 14, 9, 11, [&] {
    const HeadsArg h(a[0]);
    const Ints cb(a[10]), offs(a[11]);
    need(cb.p && offs.p && cb.n > 0 && offs.n > 0 && cb.last() == offs.n - 1 && a[5] != Py_None);
    const int64_t T = offs.last(), hq = h.h->n_q_heads, hkv = h.h->n_kv_heads, d = h.h->head_dim;
    const TensorArg q(a[1], hq, d, T), k(a[2], hkv, d, T), v(a[3], hkv, d, T), o(a[4], hq, d, T), g(a[6], hq, d, T), dq(a[7], hq, d, T),
        dk(a[8], hkv, d, T), dv(a[9], hkv, d, T);
    const float *const lse = lse_of(a[5], T, hq);
    const Workspace ws(a[12]);
    void *const stream = stream_of(a[13]);
    return unlocked([&] {
      return lib.prompts_backward(h.h, q.p, k.p, v.p, o.p, lse, g.p, dq.p, dk.p, dv.p, (int32_t)(cb.n - 1), cb.p, offs.p, ws.p, ws.bytes, stream);
    });
  });
}

// setup(Heads class, current_device(), raw_stream(device) or None, addresses of the entry points in the order of `lib`)
PyObject *setup(PyObject *, PyObject *args) {
  PyObject *type, *dev, *raw;
  unsigned long long at[7];
  if (!PyArg_ParseTuple(args, "O!OO(KKKKKKK)", &PyType_Type, &type, &dev, &raw, at, at + 1, at + 2, at + 3, at + 4, at + 5, at + 6)) return nullptr;
  Py_INCREF(type), Py_INCREF(dev), Py_INCREF(raw);
  heads_type = (PyTypeObject *)type;
  get_device = dev;
  get_raw_stream = raw == Py_None ? nullptr : raw;
  static_assert(sizeof(lib) == 7 * sizeof(void *), "an address each");
  void *p[7];
  for (int i = 0; i < 7; ++i) p[i] = (void *)(uintptr_t)at[i];
  memcpy(&lib, p, sizeof(lib));
  Py_RETURN_NONE;
}

#define FAST(name, fn) {name, (PyCFunction)(void (*)(void))(fn), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {{"setup", setup, METH_VARARGS, nullptr},
                         FAST("encode_blocks", encode_blocks),
                         FAST("reencode_positions", reencode_positions),
                         FAST("final_block", final_block<false>),
                         FAST("final_block_static", final_block<true>),
                         FAST("final_block_cached", final_block_cached),
                         FAST("prompts", prompts),
                         FAST("prompts_backward", prompts_backward),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_face", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__face() {
  import_array();
  name_c = PyUnicode_InternFromString("c");
  name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!name_c || !name_cuda_stream) return nullptr;
  PyObject *m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", TORCH_VERSION) < 0) Py_CLEAR(m);
  return m;
}
