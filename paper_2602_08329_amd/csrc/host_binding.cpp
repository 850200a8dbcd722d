// CPython extension of the binding: the marshalling of one call in native
// code.  Each function checks its tensors as binding.py does (type, dtype,
// contiguity, exact shape against the cache descriptor, the cache's GPU),
// gathers their data pointers and calls libprhs (whose entry points bind()
// receives as addresses) with the interpreter lock released.  It returns the
// library's status, or None when any check does not hold or a tensor is not a
// plain torch.Tensor: binding.py then runs its own checks, which raise, or
// make the call.  Nothing is kept from one call to the next.
//
// What it is for: a call spent 12.9 us in the Python checks and ctypes,
// longer than most decode launches take; with this it is enqueued in 4.2 us.
#include <torch/csrc/autograd/python_variable.h>

#include <initializer_list>

#include "prhs.h"

namespace {

struct Entries {
  decltype(&prhs_select) select;
  decltype(&prhs_select_shared) select_shared;
  decltype(&prhs_select_gated) select_gated;
  decltype(&prhs_gate_select) gate_select;
  decltype(&prhs_dilate_reuse) dilate_reuse;
  decltype(&prhs_sparse_decode_attn) sparse;
  decltype(&prhs_sparse_decode_attn_static) sparse_static;
  decltype(&prhs_reuse_decode_attn) reuse;
  decltype(&prhs_dense_decode_attn) dense;
  decltype(&prhs_pool_decode_attn) pool;
  decltype(&prhs_prefill_attn) prefill;
  decltype(&prhs_schedule) schedule;
} E;

// A check that does not hold: the caller answers None.
struct Slow {};

void need(bool ok) {
  if (!ok) throw Slow();
}

long long as_int(PyObject* o) {
  need(PyLong_CheckExact(o));
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) {
    PyErr_Clear();
    throw Slow();
  }
  return v;
}

int as_i32(PyObject* o) {
  const long long v = as_int(o);
  need(v >= INT32_MIN && v <= INT32_MAX);
  return (int)v;
}

double as_double(PyObject* o) {
  need(PyFloat_CheckExact(o));
  return PyFloat_AS_DOUBLE(o);
}

template <typename T>
T* as_ptr(PyObject* o) {
  return o == Py_None ? nullptr : (T*)(uintptr_t)as_int(o);
}

const at::Tensor& tensor(PyObject* o, int dev) {
  need(THPVariable_CheckExact(o));
  const at::Tensor& t = THPVariable_Unpack(o);
  need(t.defined() && t.layout() == at::kStrided && t.device().type() == at::kCUDA &&
       t.device().index() == dev);
  return t;
}

template <typename T>
T* data(PyObject* o, at::ScalarType dtype, std::initializer_list<int64_t> shape, int dev) {
  const at::Tensor& t = tensor(o, dev);
  need(t.scalar_type() == dtype && t.is_contiguous() &&
       t.sizes().equals(c10::IntArrayRef(shape.begin(), shape.size())));
  return (T*)t.data_ptr();
}

// The descriptor and its tensors, which must still be on the GPU the
// descriptor was made for.
struct Cache {
  const prhs_kv* c;
  int dev;
  int64_t b, hq, hkv, d;
  at::ScalarType dtype;
  Cache(PyObject* addr, PyObject* keep, PyObject* index) : c(as_ptr<prhs_kv>(addr)), dev(as_i32(index)) {
    need(c && dev >= 0 && PyTuple_CheckExact(keep));
    for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(keep); ++i)
      if (PyTuple_GET_ITEM(keep, i) != Py_None) tensor(PyTuple_GET_ITEM(keep, i), dev);
    b = c->batch;
    hq = c->num_q_heads;
    hkv = c->num_kv_heads;
    d = c->head_dim;
    dtype = c->dtype == PRHS_BF16 ? at::kBFloat16 : at::kFloat;
  }
  const void* q(PyObject* o) const { return data<void>(o, dtype, {b, hq, d}, dev); }
  float* out(PyObject* o) const { return data<float>(o, at::kFloat, {b, hq, d}, dev); }
  float* lse(PyObject* o) const {
    return o == Py_None ? nullptr : data<float>(o, at::kFloat, {b, hq}, dev);
  }
  int32_t* units(PyObject* o) const { return data<int32_t>(o, at::kInt, {b, hkv}, dev); }
  int32_t* flat_units(PyObject* o) const { return data<int32_t>(o, at::kInt, {b * hkv}, dev); }
  int32_t* lens(PyObject* o) const { return data<int32_t>(o, at::kInt, {b}, dev); }
  // [b][hkv][cap], cap from the tensor
  int32_t* rows(PyObject* o, int* cap) const {
    const at::Tensor& t = tensor(o, dev);
    need(t.dim() == 3 && t.size(2) <= INT32_MAX);
    *cap = (int)t.size(2);
    return data<int32_t>(o, at::kInt, {b, hkv, t.size(2)}, dev);
  }
  void* ws(PyObject* o, size_t* bytes) const {
    const at::Tensor& t = tensor(o, dev);
    need(t.dim() == 1);
    *bytes = (size_t)t.numel();
    return data<void>(o, at::kByte, {t.size(0)}, dev);
  }
};

template <typename F>
PyObject* guarded(Py_ssize_t have, Py_ssize_t want, F f) {
  try {
    need(have == want);
    return f();
  } catch (...) {  // also what torch throws on a tensor without storage
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

template <typename F>
PyObject* call(F f) {
  prhs_status st;
  Py_BEGIN_ALLOW_THREADS
  st = f();
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(st);
}

// Every function's first three arguments are the descriptor's address, its
// tensors and its GPU's index, its last the stream's handle.
#define ARGS PyObject *, PyObject *const *a, Py_ssize_t n

PyObject* f_select(ARGS) {
  return guarded(n, 11, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int kcap, scap;
    size_t wb;
    const void* q = kv.q(a[3]);
    const auto* p = as_ptr<prhs_params>(a[4]);
    int32_t *ti = kv.rows(a[5], &kcap), *tl = kv.units(a[6]), *si = kv.rows(a[7], &scap), *sl = kv.units(a[8]);
    void* ws = kv.ws(a[9], &wb);
    void* st = as_ptr<void>(a[10]);
    return call([&] { return E.select(kv.c, q, p, ti, tl, kcap, si, sl, scap, ws, wb, st); });
  });
}

PyObject* f_select_shared(ARGS) {
  return guarded(n, 13, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int kcap, scap, hcap;
    size_t wb;
    const void* q = kv.q(a[3]);
    const auto* p = as_ptr<prhs_params>(a[4]);
    int32_t *ti = kv.rows(a[5], &kcap), *tl = kv.units(a[6]), *si = kv.rows(a[7], &scap), *sl = kv.units(a[8]);
    int32_t *hi = kv.rows(a[9], &hcap), *hl = kv.units(a[10]);
    need(hcap == scap);
    void* ws = kv.ws(a[11], &wb);
    void* st = as_ptr<void>(a[12]);
    return call([&] { return E.select_shared(kv.c, q, p, ti, tl, kcap, si, sl, scap, hi, hl, ws, wb, st); });
  });
}

PyObject* f_select_gated(ARGS) {
  return guarded(n, 14, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int kcap, scap, hcap;
    size_t wb;
    const void* q = kv.q(a[3]);
    const auto* p = as_ptr<prhs_params>(a[4]);
    const int32_t* choice = kv.flat_units(a[5]);
    int32_t *ti = kv.rows(a[6], &kcap), *tl = kv.units(a[7]), *si = kv.rows(a[8], &scap), *sl = kv.units(a[9]);
    int32_t *hi = kv.rows(a[10], &hcap), *hl = kv.units(a[11]);
    need(hcap == scap);
    void* ws = kv.ws(a[12], &wb);
    void* st = as_ptr<void>(a[13]);
    return call([&] { return E.select_gated(kv.c, q, p, choice, ti, tl, kcap, si, sl, scap, hi, hl, ws, wb, st); });
  });
}

PyObject* f_gate_select(ARGS) {
  return guarded(n, 22, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int kcap, scap, hcap;
    size_t wb;
    const void* q = kv.q(a[3]);
    const auto* p = as_ptr<prhs_params>(a[4]);
    const double tau = as_double(a[5]);
    const int slot = as_i32(a[6]);
    const at::Tensor& r = tensor(a[7], kv.dev);
    need(r.dim() == 4 && r.size(0) <= INT32_MAX);
    const int64_t S = r.size(0), U = kv.b * kv.hkv;
    void* ref = data<void>(a[7], kv.dtype, {S, kv.b, kv.hq, kv.d}, kv.dev);
    int32_t* valid = data<int32_t>(a[8], at::kInt, {S, U}, kv.dev);
    int32_t* slens = data<int32_t>(a[9], at::kInt, {S, kv.b}, kv.dev);
    int32_t *choice = kv.flat_units(a[10]), *ra = kv.flat_units(a[11]), *ro = kv.flat_units(a[12]),
            *tail = kv.flat_units(a[13]);
    int32_t *ti = kv.rows(a[14], &kcap), *tl = kv.units(a[15]), *si = kv.rows(a[16], &scap), *sl = kv.units(a[17]);
    int32_t *hi = kv.rows(a[18], &hcap), *hl = kv.units(a[19]);
    need(hcap == scap);
    void* ws = kv.ws(a[20], &wb);
    void* st = as_ptr<void>(a[21]);
    return call([&] {
      return E.gate_select(kv.c, q, p, tau, (int)S, slot, ref, valid, slens, choice, ra, ro, tail, ti, tl,
                           kcap, si, sl, scap, hi, hl, ws, wb, st);
    });
  });
}

PyObject* f_dilate_reuse(ARGS) {  // no descriptor: params, the six arrays, the stream
  return guarded(n, 8, [&] {
    const auto* p = as_ptr<prhs_params>(a[0]);
    need(THPVariable_CheckExact(a[1]));
    const at::Tensor& t = THPVariable_Unpack(a[1]);
    const int dev = t.device().index();
    need(t.dim() == 3 && t.size(0) <= INT32_MAX && t.size(1) <= INT32_MAX && t.size(2) <= INT32_MAX);
    const int64_t b = t.size(0), h = t.size(1);
    const int32_t* ti = data<int32_t>(a[1], at::kInt, {b, h, t.size(2)}, dev);
    const int32_t* tl = data<int32_t>(a[2], at::kInt, {b, h}, dev);
    const int32_t* al = data<int32_t>(a[3], at::kInt, {b}, dev);
    const int32_t* sl = data<int32_t>(a[4], at::kInt, {b}, dev);
    const at::Tensor& s = tensor(a[5], dev);
    need(s.dim() == 3 && s.size(2) <= INT32_MAX);
    int32_t* si = data<int32_t>(a[5], at::kInt, {b, h, s.size(2)}, dev);
    int32_t* sn = data<int32_t>(a[6], at::kInt, {b, h}, dev);
    const int kcap = (int)t.size(2), scap = (int)s.size(2);
    void* st = as_ptr<void>(a[7]);
    return call([&] { return E.dilate_reuse(p, (int)b, (int)h, ti, tl, kcap, al, sl, si, sn, scap, st); });
  });
}

PyObject* f_sparse(ARGS) {  // without a workspace (None): the static form
  return guarded(n, 11, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int cap;
    size_t wb = 0;
    const void* q = kv.q(a[3]);
    const int32_t *si = kv.rows(a[4], &cap), *sl = kv.units(a[5]);
    const float scale = (float)as_double(a[6]);
    float *out = kv.out(a[7]), *lse = kv.lse(a[8]);
    void* ws = a[9] == Py_None ? nullptr : kv.ws(a[9], &wb);
    const bool fixed = a[9] == Py_None;
    void* st = as_ptr<void>(a[10]);
    return call([&] {
      return fixed ? E.sparse_static(kv.c, q, si, sl, cap, scale, out, lse, st)
                   : E.sparse(kv.c, q, si, sl, cap, scale, out, lse, ws, wb, st);
    });
  });
}

PyObject* f_reuse(ARGS) {
  return guarded(n, 12, [&] {
    const Cache kv(a[0], a[1], a[2]);
    int cap;
    size_t wb;
    const void* q = kv.q(a[3]);
    const int32_t *si = kv.rows(a[4], &cap), *sl = kv.units(a[5]), *al = kv.lens(a[6]);
    const float scale = (float)as_double(a[7]);
    float *out = kv.out(a[8]), *lse = kv.lse(a[9]);
    void* ws = kv.ws(a[10], &wb);
    void* st = as_ptr<void>(a[11]);
    return call([&] { return E.reuse(kv.c, q, si, sl, cap, al, scale, out, lse, ws, wb, st); });
  });
}

PyObject* f_dense(ARGS) {
  return guarded(n, 9, [&] {
    const Cache kv(a[0], a[1], a[2]);
    size_t wb;
    const void* q = kv.q(a[3]);
    const float scale = (float)as_double(a[4]);
    float *out = kv.out(a[5]), *lse = kv.lse(a[6]);
    void* ws = kv.ws(a[7], &wb);
    void* st = as_ptr<void>(a[8]);
    return call([&] { return E.dense(kv.c, q, scale, out, lse, ws, wb, st); });
  });
}

PyObject* f_pool(ARGS) {
  return guarded(n, 16, [&] {
    const Cache kv(a[0], a[1], a[2]);
    size_t wb;
    const void* q = kv.q(a[3]);
    const at::Tensor& p = tensor(a[4], kv.dev);
    need(p.scalar_type() == at::kInt && p.is_contiguous() && p.dim() >= 1 && p.size(-1) >= 1 &&
         p.size(-1) <= INT32_MAX && p.numel() / p.size(-1) <= INT32_MAX);
    const at::Tensor& pl = tensor(a[5], kv.dev);
    need(pl.scalar_type() == at::kInt && pl.is_contiguous() &&
         pl.sizes().equals(p.sizes().slice(0, p.dim() - 1)));
    const int cap = (int)p.size(-1), rows = (int)(p.numel() / p.size(-1));
    const int32_t *ur = kv.flat_units(a[6]), *ut = kv.flat_units(a[7]);
    const int side = as_i32(a[9]);
    const int32_t* gate = nullptr;
    if (side != PRHS_UNITS_ALL) gate = kv.flat_units(a[8]);
    else if (a[8] != Py_None) tensor(a[8], kv.dev);
    const auto* ps = as_ptr<prhs_psaw>(a[10]);
    const float scale = (float)as_double(a[11]);
    float *out = kv.out(a[12]), *lse = kv.lse(a[13]);
    void* ws = kv.ws(a[14], &wb);
    void* st = as_ptr<void>(a[15]);
    const auto *pi = (const int32_t*)p.data_ptr(), *pn = (const int32_t*)pl.data_ptr();
    return call([&] {
      return E.pool(kv.c, q, pi, pn, rows, cap, ur, ut, gate, side, ps, scale, out, lse, ws, wb, st);
    });
  });
}

PyObject* f_prefill(ARGS) {
  return guarded(n, 9, [&] {
    const Cache kv(a[0], a[1], a[2]);
    const at::Tensor& t = tensor(a[3], kv.dev);
    need(t.dim() == 4 && t.size(2) <= INT32_MAX);
    const int64_t T = t.size(2);
    const void* q = data<void>(a[3], kv.dtype, {kv.b, kv.hq, T, kv.d}, kv.dev);
    const float scale = (float)as_double(a[4]);
    float* out = data<float>(a[5], at::kFloat, {kv.b, kv.hq, T, kv.d}, kv.dev);
    float* lse = a[6] == Py_None ? nullptr : data<float>(a[6], at::kFloat, {kv.b, kv.hq, T}, kv.dev);
    const auto* ps = as_ptr<prhs_psaw>(a[7]);
    void* st = as_ptr<void>(a[8]);
    return call([&] { return E.prefill(kv.c, q, (int)T, ps, scale, out, lse, st); });
  });
}

PyObject* f_schedule(ARGS) {  // the library's answer, -1 included
  return guarded(n, 3, [&] {
    return PyLong_FromLong(E.schedule(as_i32(a[0]), as_i32(a[1]), as_ptr<prhs_params>(a[2])));
  });
}

// bind(addresses): the library's entry points, in the order of Entries.
PyObject* f_bind(ARGS) {
  constexpr Py_ssize_t kEntries = sizeof(Entries) / sizeof(void*);
  if (n != kEntries) {
    PyErr_Format(PyExc_TypeError, "bind takes %zd addresses", kEntries);
    return nullptr;
  }
  Entries e;
  for (Py_ssize_t i = 0; i < n; ++i) {
    void* p = PyLong_AsVoidPtr(a[i]);
    if (!p) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "a null address");
      return nullptr;
    }
    ((void**)&e)[i] = p;
  }
  E = e;
  Py_RETURN_NONE;
}

#define FAST(name) {#name, (PyCFunction)(void (*)(void))f_##name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {
    FAST(bind), FAST(select), FAST(select_shared), FAST(select_gated), FAST(gate_select),
    FAST(dilate_reuse), FAST(sparse), FAST(reuse), FAST(dense), FAST(pool), FAST(prefill),
    FAST(schedule), {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_prhs_host", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

// torch_version and abi_version: what this was compiled against, for the
// binding to compare with what is loaded.
PyMODINIT_FUNC PyInit__prhs_host() {
  PyObject* m = PyModule_Create(&module);
  if (m && (PyModule_AddStringConstant(m, "torch_version", PRHS_TORCH_VERSION) < 0 ||
            PyModule_AddIntConstant(m, "abi_version", PRHS_ABI_VERSION) < 0))
    Py_CLEAR(m);
  return m;
}
