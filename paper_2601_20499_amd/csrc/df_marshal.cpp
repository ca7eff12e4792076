// Python extension `_marshal`: the binding's calls that a generation loop makes for every layer, with their arguments taken from
// torch tensors and lists of whole numbers in native code.  In Python an attention call's arguments took 5.4 us, as long as the whole
// launch of 64 queries, and those of an append 2.4 us.
//
// A function returns the library's status (a pack also its two lists), or None for anything but the ordinary kinds of arguments -
// exact torch.Tensor objects on a GPU, lists or tuples of int that fit the C type, a float, a stream given as int
// or not at all - or for sizes that do not go together: then nothing has been called, and binding.py takes the arguments
// its own way, with its own errors.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "df.h"

namespace {

decltype(&df_attn_fwd) attn_fwd, attn_fwd_static;
decltype(&df_head_score) head_score;
decltype(&df_kv_append) kv_append;
decltype(&df_pack_context) pack_context;

// The readers below say whether an argument is of the ordinary kind.  (Nothing is thrown where it is not: that took 3 to 5 us, a third to a half of
// what a call costs that is marshalled in Python, such as one with a torch.cuda.Stream.)
const at::Tensor *tensor(PyObject *x) {
  if (!THPVariable_CheckExact(x)) return nullptr;
  const at::Tensor &t = THPVariable_Unpack(x);
  return t.is_cuda() ? &t : nullptr;
}
const at::Tensor *tensor(PyObject *x, int64_t dims) {
  const at::Tensor *t = tensor(x);
  return t && t->dim() == dims ? t : nullptr;
}
void *address(const at::Tensor &t) { return t.numel() == 0 ? nullptr : t.data_ptr(); }
template <class T>
bool address_or_null(PyObject *x, T *&to) {
  to = nullptr;
  if (x == Py_None) return true;
  const at::Tensor *t = tensor(x);
  if (t) to = static_cast<T *>(address(*t));
  return t != nullptr;
}
bool buffer_or_null(PyObject *x, void *&to, size_t &bytes) {
  to = nullptr;
  bytes = 0;
  if (x == Py_None) return true;
  const at::Tensor *t = tensor(x);
  if (t == nullptr) return false;
  to = address(*t);
  bytes = size_t(t->numel()) * t->element_size();
  return true;
}
bool size32(int64_t n, int32_t &to) {
  to = int32_t(n);
  return n <= INT32_MAX;
}

// A list or tuple of whole numbers as a C array of at least `at_least` of them.
template <class T>
struct Numbers {
  T at[2 * DF_MAX_HEADS];
  bool read(PyObject *x, Py_ssize_t at_least) {
    if (!PyList_CheckExact(x) && !PyTuple_CheckExact(x)) return false;
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(x);
    if (n < at_least || n > 2 * DF_MAX_HEADS) return false;
    PyObject **items = PySequence_Fast_ITEMS(x);
    for (Py_ssize_t i = 0; i < n; ++i) {
      if (!PyLong_CheckExact(items[i])) return false;
      int overflow = 0;
      const long long v = PyLong_AsLongLongAndOverflow(items[i], &overflow);
      at[i] = T(v);
      if (overflow || at[i] != v) return false;
    }
    return true;
  }
  // None: no list.
  template <class P>
  bool read_or_null(PyObject *x, Py_ssize_t at_least, P *&to) {
    to = nullptr;
    if (x == Py_None) return true;
    to = at;
    return read(x, at_least);
  }
};
bool number(PyObject *x, int32_t &to) {
  if (!PyLong_CheckExact(x)) return false;
  int overflow = 0;
  const long v = PyLong_AsLongAndOverflow(x, &overflow);
  to = int32_t(v);
  return !overflow && to == v;
}
bool real(PyObject *x, float &to) {
  if (!PyFloat_CheckExact(x)) return false;
  to = float(PyFloat_AS_DOUBLE(x));
  return true;
}
// None: the current stream of the current device.
bool stream(PyObject *x, void *&to) {
  if (x == Py_None) {
    to = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  if (!PyLong_CheckExact(x)) return false;
  to = PyLong_AsVoidPtr(x);
  if (to != nullptr || !PyErr_Occurred()) return true;
  PyErr_Clear();
  return false;
}

template <class Call>
df_status without_gil(Call &&call) {
  df_status s;
  Py_BEGIN_ALLOW_THREADS
  s = call();
  Py_END_ALLOW_THREADS
  return s;
}
// The C struct of a binding.Cache, or null.
struct CacheOf {
  Py_buffer view{};
  df_cache *cache = nullptr;
  explicit CacheOf(PyObject *x) {
    PyObject *c = PyObject_GetAttrString(x, "c");
    if (c == nullptr || PyObject_GetBuffer(c, &view, PyBUF_WRITABLE) != 0) PyErr_Clear();
    else if (size_t(view.len) == sizeof(df_cache)) cache = static_cast<df_cache *>(view.buf);
    Py_XDECREF(c);                   // the view holds it
    if (cache && (cache->H < 0 || cache->H > DF_MAX_HEADS)) cache = nullptr;
  }
  CacheOf(const CacheOf &) = delete;
  ~CacheOf() { PyBuffer_Release(&view); }          // nothing where there is no view
};

// Runs `body`; null without a Python error, and what torch throws for a tensor that has no address, is None.
template <class Body>
PyObject *or_none(Py_ssize_t n, Py_ssize_t wanted, Body &&body) {
  if (n == wanted) {
    try {
      PyObject *result = body();
      if (result != nullptr || PyErr_Occurred()) return result;
    } catch (const std::exception &) {
    }
  }
  Py_RETURN_NONE;
}

// q, k_cur, v_cur, k_hist, v_hist, hist_off, hist_sink_len, out, softmax_scale, lse_out, score_out, workspace, stream, hist_len, static
PyObject *attn(PyObject *, PyObject *const *x, Py_ssize_t n) {
  return or_none(n, 15, [&]() -> PyObject * {
    const at::Tensor *q = tensor(x[0], 3), *k = tensor(x[1], 3), *v = tensor(x[2]), *out = tensor(x[7], 3);
    df_attn_args a{};
    void *st;
    Numbers<int64_t> off;
    Numbers<int32_t> sink, len;
    if (!q || !k || !v || !out || !stream(x[12], st) || !real(x[8], a.softmax_scale) || v->strides() != k->strides() ||
        !size32(q->size(1), a.H) || !size32(q->size(2), a.d) || !size32(q->size(0), a.Nq) || !size32(k->size(0), a.Nc) ||
        !off.read(x[5], Py_ssize_t(a.H) + 1) || !sink.read_or_null(x[6], a.H, a.hist_sink_len) ||
        !len.read_or_null(x[13], a.H, a.hist_len) || !address_or_null(x[3], a.k_hist) || !address_or_null(x[4], a.v_hist) ||
        !address_or_null(x[9], a.lse_out) || !address_or_null(x[10], a.score_out) ||
        !buffer_or_null(x[11], a.workspace, a.workspace_bytes))
      return nullptr;
    a.q = address(*q);
    a.q_stride_tok = q->stride(0);
    a.q_stride_head = q->stride(1);
    a.k_cur = address(*k);
    a.v_cur = address(*v);
    a.kc_stride_tok = k->stride(0);
    a.kc_stride_head = k->stride(1);
    a.hist_off = off.at;
    a.out = address(*out);
    a.o_stride_tok = out->stride(0);
    a.o_stride_head = out->stride(1);
    const auto entry = x[14] == Py_True ? attn_fwd_static : attn_fwd;
    return PyLong_FromLong(without_gil([&] { return entry(&a, st); }));
  });
}

// q, k_cur, k_hist, hist_off, hist_sink_len, score_out, softmax_scale, q_sample_stride, q_offset, workspace, stream, hist_len
PyObject *score(PyObject *, PyObject *const *x, Py_ssize_t n) {
  return or_none(n, 12, [&]() -> PyObject * {
    const at::Tensor *q = tensor(x[0], 3), *k = tensor(x[1], 3);
    df_score_args a{};
    void *st;
    Numbers<int64_t> off;
    Numbers<int32_t> sink, len;
    if (!q || !k || !stream(x[10], st) || !real(x[6], a.softmax_scale) || !number(x[7], a.q_sample_stride) || !number(x[8], a.q_offset) ||
        !size32(q->size(1), a.H) || !size32(q->size(2), a.d) || !size32(q->size(0), a.Nq) || !size32(k->size(0), a.Nc) ||
        !off.read(x[3], Py_ssize_t(a.H) + 1) || !sink.read(x[4], a.H) || !len.read_or_null(x[11], a.H, a.hist_len) ||
        !address_or_null(x[2], a.k_hist) || !address_or_null(x[5], a.score_out) ||
        !buffer_or_null(x[9], a.workspace, a.workspace_bytes))
      return nullptr;
    a.q = address(*q);
    a.q_stride_tok = q->stride(0);
    a.q_stride_head = q->stride(1);
    a.k_cur = address(*k);
    a.kc_stride_tok = k->stride(0);
    a.kc_stride_head = k->stride(1);
    a.hist_off = off.at;
    a.hist_sink_len = sink.at;
    return PyLong_FromLong(without_gil([&] { return head_score(&a, st); }));
  });
}

// cache, k_new, v_new, stream
PyObject *append(PyObject *, PyObject *const *x, Py_ssize_t n) {
  return or_none(n, 4, [&]() -> PyObject * {
    const at::Tensor *k = tensor(x[1], 3), *v = tensor(x[2]);
    df_append_args a{};
    void *st;
    if (!k || !v || !stream(x[3], st) || v->strides() != k->strides() || !size32(k->size(0), a.Nc)) return nullptr;
    const CacheOf cache(x[0]);
    if (!cache.cache) return nullptr;
    a.cache = cache.cache;
    a.k_new = address(*k);
    a.v_new = address(*v);
    a.stride_tok = k->stride(0);
    a.stride_head = k->stride(1);
    return PyLong_FromLong(without_gil([&] { return kv_append(&a, st); }));
  });
}

template <class T>
PyObject *list_of(const T *x, int n) {
  PyObject *list = PyList_New(n);
  for (int i = 0; list && i < n; ++i) {
    PyObject *v = PyLong_FromLongLong(x[i]);
    if (v == nullptr) {
      Py_DECREF(list);
      return nullptr;
    }
    PyList_SET_ITEM(list, i, v);
  }
  return list;
}
// cache, take_sink, take_win, k_out, v_out, stream -> status, hist_off, sink_len
PyObject *pack(PyObject *, PyObject *const *x, Py_ssize_t n) {
  return or_none(n, 6, [&]() -> PyObject * {
    const at::Tensor *k = tensor(x[3]), *v = tensor(x[4]);
    void *st;
    if (!k || !v || k->dim() < 1 || !stream(x[5], st)) return nullptr;
    const CacheOf cache(x[0]);
    if (!cache.cache) return nullptr;
    const int H = cache.cache->H;
    Numbers<int32_t> sink, win;
    if (!sink.read(x[1], H) || !win.read(x[2], H)) return nullptr;
    int64_t off[DF_MAX_HEADS + 1] = {};
    int32_t sink_len[DF_MAX_HEADS] = {};
    df_pack_args a{};
    a.cache = cache.cache;
    a.take_sink = sink.at;
    a.take_win = win.at;
    a.k_out = address(*k);
    a.v_out = address(*v);
    a.out_capacity_rows = k->size(0);
    a.hist_off_out = off;
    a.sink_len_out = sink_len;
    const df_status s = without_gil([&] { return pack_context(&a, st); });
    PyObject *o = list_of(off, H + 1), *l = o ? list_of(sink_len, H) : nullptr;
    if (l == nullptr) {
      Py_XDECREF(o);
      return nullptr;
    }
    return Py_BuildValue("iNN", int(s), o, l);
  });
}

// Addresses of df_attn_fwd, df_attn_fwd_static, df_head_score, df_kv_append and df_pack_context in the library that the binding loaded.
PyObject *setup(PyObject *, PyObject *const *x, Py_ssize_t n) {
  void *f[5];
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "five addresses");
    return nullptr;
  }
  for (int i = 0; i < 5; ++i) {
    f[i] = PyLong_AsVoidPtr(x[i]);
    if (f[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a function has no address");
      return nullptr;
    }
  }
  attn_fwd = reinterpret_cast<decltype(attn_fwd)>(f[0]);
  attn_fwd_static = reinterpret_cast<decltype(attn_fwd_static)>(f[1]);
  head_score = reinterpret_cast<decltype(head_score)>(f[2]);
  kv_append = reinterpret_cast<decltype(kv_append)>(f[3]);
  pack_context = reinterpret_cast<decltype(pack_context)>(f[4]);
  Py_RETURN_NONE;
}

template <class F>
PyCFunction as_c(F f) { return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)); }
PyMethodDef methods[] = {{"setup", as_c(setup), METH_FASTCALL, nullptr},   {"attn", as_c(attn), METH_FASTCALL, nullptr},
                         {"score", as_c(score), METH_FASTCALL, nullptr},   {"append", as_c(append), METH_FASTCALL, nullptr},
                         {"pack", as_c(pack), METH_FASTCALL, nullptr},     {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() { return PyModule_Create(&module); }
