// Native marshalling for the calls a decode step or a small compression makes: from torch tensors to the C ABI's
// layouts and pointers without a Python object per field (a call of the ctypes route builds a dozen and takes 10 to
// 17 us, as long as the kernels of a short cache run; these take 2 to 4, the launch included).
//
// Each function takes the well-formed case only: tensors of the plain class on a GPU, outputs and workspace given,
// numbers in range.  It returns the library's status, or None for anything else - the caller then takes the
// ctypes route, which handles or refuses it.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/core/TensorBase.h>
#include <torch/csrc/autograd/python_variable.h>

#include "ckv.h"

namespace {

struct Entry {
  decltype(&ckv_compress) compress;
  decltype(&ckv_append) append;
  decltype(&ckv_decode_attn) decode_attn;
  decltype(&ckv_paged_append) paged_append;
  decltype(&ckv_paged_decode_attn) paged_decode_attn;
} entry;

// a tensor argument: NULL for None; `ok` turns false for what this file does not take
const at::TensorBase* tensor(PyObject* x, bool& ok) {
  if (x == Py_None) return nullptr;
  if (!THPVariable_CheckExact(x)) { ok = false; return nullptr; }
  const at::TensorBase& t = THPVariable_Unpack(x);
  if (!t.is_cuda() || t.layout() != at::kStrided) { ok = false; return nullptr; }
  return &t;
}
const at::TensorBase* given(PyObject* x, bool& ok) {
  const at::TensorBase* t = tensor(x, ok);
  if (!t) ok = false;
  return t;
}
template <typename T = void>
T* ptr(const at::TensorBase* t) { return t ? static_cast<T*>(t->data_ptr()) : nullptr; }

int32_t small_int(PyObject* x, bool& ok) {
  if (!PyLong_CheckExact(x)) { ok = false; return 0; }
  int over = 0;
  const long long v = PyLong_AsLongLongAndOverflow(x, &over);
  if (over || v < INT32_MIN || v > INT32_MAX) { ok = false; return 0; }
  return (int32_t)v;
}
float number(PyObject* x, bool& ok) {
  if (PyFloat_CheckExact(x)) return (float)PyFloat_AS_DOUBLE(x);
  return (float)small_int(x, ok);
}
void* stream(PyObject* x) { return PyLong_AsVoidPtr(x); }   // the caller's own number

int dtype_of(const at::TensorBase& t, bool& ok) {
  if (t.scalar_type() == at::kFloat) return CKV_F32;
  if (t.scalar_type() == at::kBFloat16) return CKV_BF16;
  ok = false;
  return 0;
}
int32_t fits(int64_t v, bool& ok) {
  if (v < 0 || v > INT32_MAX) ok = false;
  return (int32_t)v;
}

// what layout_of() makes of a cache tensor and its degrees
ckv_layout layout(const at::TensorBase& t, const at::TensorBase* deg, bool& ok) {
  ckv_layout l{};
  if (t.dim() != 4) { ok = false; return l; }
  const auto n = t.sizes(), s = t.strides();
  l.dtype = dtype_of(t, ok);
  if (s[3] != 1) ok = false;
  l.batch = fits(n[0], ok); l.heads = fits(n[1], ok); l.seq = fits(n[2], ok); l.dim = fits(n[3], ok);
  l.stride_b = s[0]; l.stride_h = s[1]; l.stride_s = s[2];
  if (deg) {
    if (deg->scalar_type() != at::kInt || deg->dim() != 3 || deg->size(0) != n[0] || deg->size(1) != n[1] ||
        deg->size(2) != n[2] || (n[2] > 1 && deg->stride(2) != 1))
      ok = false;
    else {
      const auto d = deg->strides();
      l.deg_stride = n[1] > 1 ? d[1] : n[0] > 1 ? d[0] : n[2];
      if (n[0] > 1 && n[1] > 1 && d[0] != n[1] * d[1]) ok = false;
    }
  }
  return l;
}
bool rows_of(const at::TensorBase& t, int64_t b, int64_t h, int64_t d, at::ScalarType type) {
  return t.dim() == 3 && t.size(0) == b && t.size(1) == h && t.size(2) == d && t.is_contiguous() && t.scalar_type() == type;
}
ckv_paged_layout paged(const at::TensorBase& pool, const at::TensorBase& table, bool& ok) {
  ckv_paged_layout l{};
  if (pool.dim() != 4 || !pool.is_contiguous() || table.dim() != 2 || table.scalar_type() != at::kInt || !table.is_contiguous()) {
    ok = false;
    return l;
  }
  l.batch = fits(table.size(0), ok); l.heads = fits(pool.size(1), ok); l.dim = fits(pool.size(3), ok);
  l.dtype = dtype_of(pool, ok); l.block_size = fits(pool.size(2), ok); l.max_blocks = fits(table.size(1), ok);
  l.n_blocks = fits(pool.size(0), ok);
  return l;
}

// Counts the arguments, runs `body` (ok may turn false at any point) and turns its status into a Python number.
template <typename F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F&& body) {
  if (n != want) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  bool ok = true;
  int status = 0;
  try {
    status = body(ok);
  } catch (...) {              // (a tensor without storage and the like: the ctypes route reports it)
    ok = false;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  if (!ok) Py_RETURN_NONE;
  return PyLong_FromLong(status);
}
template <typename F>
int unlocked(F&& call) {
  int status;
  Py_BEGIN_ALLOW_THREADS
  status = call();
  Py_END_ALLOW_THREADS
  return status;
}

// K, V, deg, chunk, retain_ratio, rounds, n_sink, n_recent, scope, flags, K_out, V_out, deg_out, assign, workspace, stream
PyObject* compress(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 16, [&](bool& ok) -> int {
    const auto *K = given(a[0], ok), *V = given(a[1], ok), *deg = tensor(a[2], ok);
    const auto *oK = given(a[10], ok), *oV = given(a[11], ok), *od = given(a[12], ok), *assign = tensor(a[13], ok);
    const auto* ws = given(a[14], ok);
    ckv_params p{};
    p.chunk = small_int(a[3], ok);
    p.retain_ratio = number(a[4], ok);
    p.n_sink = small_int(a[6], ok);
    p.n_recent = small_int(a[7], ok);
    p.scope = small_int(a[8], ok);
    p.flags = (uint32_t)small_int(a[9], ok);
    if (a[5] != Py_None) {
      if (!PyList_CheckExact(a[5])) ok = false;
      else {
        const Py_ssize_t m = PyList_GET_SIZE(a[5]);
        if (m < 1 || m > CKV_MAX_ROUNDS) ok = false;
        else for (Py_ssize_t j = 0; j < m; ++j) p.r[j] = number(PyList_GET_ITEM(a[5], j), ok);
        p.n_rounds = (int32_t)m;
      }
    }
    if (!ok) return 0;
    const ckv_layout in = layout(*K, deg, ok), out = layout(*oK, od, ok);
    (void)layout(*V, nullptr, ok);
    if (!ok || V->scalar_type() != K->scalar_type() || V->sizes() != K->sizes()) { ok = false; return 0; }
    void *k = ptr(K), *v = ptr(V), *ok_p = ptr(oK), *ov = ptr(oV), *w = ptr(ws);
    const int32_t* d = ptr<int32_t>(deg);
    int32_t *dout = ptr<int32_t>(od), *as = ptr<int32_t>(assign);
    const size_t nw = (size_t)ws->numel();
    void* s = stream(a[15]);
    return unlocked([&] { return entry.compress(k, v, d, &in, &p, ok_p, ov, dout, &out, as, w, nw, s); });
  });
}

// k_new, v_new, K, V, deg, lens, pos, stream
PyObject* append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&](bool& ok) -> int {
    const auto *kn = given(a[0], ok), *vn = given(a[1], ok), *K = given(a[2], ok), *V = given(a[3], ok);
    const auto *deg = tensor(a[4], ok), *lens = tensor(a[5], ok);
    const int32_t pos = small_int(a[6], ok);
    if (!ok) return 0;
    const ckv_layout l = layout(*K, deg, ok);
    (void)layout(*V, nullptr, ok);
    if (!ok || !rows_of(*kn, l.batch, l.heads, l.dim, K->scalar_type()) || !rows_of(*vn, l.batch, l.heads, l.dim, K->scalar_type()) ||
        V->sizes() != K->sizes() || V->strides() != K->strides()) {
      ok = false;
      return 0;
    }
    void *k1 = ptr(kn), *v1 = ptr(vn), *k = ptr(K), *v = ptr(V), *s = stream(a[7]);
    int32_t *d = ptr<int32_t>(deg), *ls = ptr<int32_t>(lens);
    return unlocked([&] { return entry.append(k1, v1, k, v, d, &l, ls, pos, s); });
  });
}

// q, K, V, lens, deg, scale, out, workspace, stream
PyObject* decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 9, [&](bool& ok) -> int {
    const auto *q = given(a[0], ok), *K = given(a[1], ok), *V = given(a[2], ok), *lens = tensor(a[3], ok), *deg = tensor(a[4], ok);
    const auto *out = given(a[6], ok), *ws = given(a[7], ok);
    const float scale = number(a[5], ok);
    if (!ok) return 0;
    const ckv_layout l = layout(*K, deg, ok);
    const int o_type = dtype_of(*out, ok);
    if (!ok || q->dim() != 3 || !q->is_contiguous() || q->scalar_type() != K->scalar_type()) { ok = false; return 0; }
    const int32_t heads = fits(q->size(1), ok);
    void *qp = ptr(q), *k = ptr(K), *v = ptr(V), *o = ptr(out), *w = ptr(ws), *s = stream(a[8]);
    const int32_t *d = ptr<int32_t>(deg), *ls = ptr<int32_t>(lens);
    const size_t nw = (size_t)ws->numel();
    return unlocked([&] { return entry.decode_attn(qp, heads, k, v, &l, ls, d, scale, o, o_type, w, nw, s); });
  });
}

// k_new, v_new, K_pool, V_pool, deg_pool, block_table, lens, stream
PyObject* paged_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 8, [&](bool& ok) -> int {
    const auto *kn = given(a[0], ok), *vn = given(a[1], ok), *K = given(a[2], ok), *V = given(a[3], ok);
    const auto *deg = tensor(a[4], ok), *table = given(a[5], ok), *lens = given(a[6], ok);
    if (!ok) return 0;
    const ckv_paged_layout l = paged(*K, *table, ok);
    if (!ok || !rows_of(*kn, l.batch, l.heads, l.dim, K->scalar_type()) || !rows_of(*vn, l.batch, l.heads, l.dim, K->scalar_type())) {
      ok = false;
      return 0;
    }
    void *k1 = ptr(kn), *v1 = ptr(vn), *k = ptr(K), *v = ptr(V), *s = stream(a[7]);
    int32_t *d = ptr<int32_t>(deg), *ls = ptr<int32_t>(lens);
    const int32_t* t = ptr<int32_t>(table);
    return unlocked([&] { return entry.paged_append(k1, v1, k, v, d, t, ls, &l, s); });
  });
}

// q, K_pool, V_pool, deg_pool, block_table, lens, max_len, scale, out, workspace, stream
PyObject* paged_decode_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&](bool& ok) -> int {
    const auto *q = given(a[0], ok), *K = given(a[1], ok), *V = given(a[2], ok), *deg = tensor(a[3], ok);
    const auto *table = given(a[4], ok), *lens = given(a[5], ok), *out = given(a[8], ok), *ws = given(a[9], ok);
    const int32_t max_len = small_int(a[6], ok);
    const float scale = number(a[7], ok);
    if (!ok) return 0;
    const ckv_paged_layout l = paged(*K, *table, ok);
    const int o_type = dtype_of(*out, ok);
    if (!ok || q->dim() != 3 || !q->is_contiguous() || q->scalar_type() != K->scalar_type()) { ok = false; return 0; }
    const int32_t heads = fits(q->size(1), ok);
    void *qp = ptr(q), *k = ptr(K), *v = ptr(V), *o = ptr(out), *w = ptr(ws), *s = stream(a[10]);
    const int32_t *d = ptr<int32_t>(deg), *ls = ptr<int32_t>(lens), *t = ptr<int32_t>(table);
    const size_t nw = (size_t)ws->numel();
    return unlocked([&] { return entry.paged_decode_attn(qp, heads, k, v, d, t, ls, &l, max_len, scale, o, o_type, w, nw, s); });
  });
}

// the addresses of the library's entry points, in Entry's order
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  if (n != 5) {
    PyErr_SetString(PyExc_TypeError, "five addresses");
    return nullptr;
  }
  void* p[5];
  for (int i = 0; i < 5; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  entry.compress = reinterpret_cast<decltype(&ckv_compress)>(p[0]);
  entry.append = reinterpret_cast<decltype(&ckv_append)>(p[1]);
  entry.decode_attn = reinterpret_cast<decltype(&ckv_decode_attn)>(p[2]);
  entry.paged_append = reinterpret_cast<decltype(&ckv_paged_append)>(p[3]);
  entry.paged_decode_attn = reinterpret_cast<decltype(&ckv_paged_decode_attn)>(p[4]);
  Py_RETURN_NONE;
}

#define CKV_METHOD(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CKV_METHOD(bind), CKV_METHOD(compress), CKV_METHOD(append), CKV_METHOD(decode_attn),
                         CKV_METHOD(paged_append), CKV_METHOD(paged_decode_attn), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_ckv_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ckv_binding(void) { return PyModule_Create(&module); }
