// Native form of the Python entry points a program calls per step (attn_fwd,
// attn_fwd_bwd, attn_bwd, attn_decode): argument checks, output and workspace
// allocation and the call into the library, without per-argument Python work.
//
// Each function answers NotImplemented, having done nothing, for anything but
// plain arguments that pass every check (tensors of exactly torch.Tensor, dense,
// on one GPU, contiguous, of matching types and shapes; numbers of exactly int,
// float or bool). The Python form then runs, with its full checks and errors.
// A status code of the library other than 0 is answered as an int.
//
// The library is reached through the addresses that bind() receives, so both
// forms call the same loaded library.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/TensorSubclassLikeUtils.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cmath>

namespace {

using WsFn = size_t (*)(int, int, int, int);
using DecWsFn = size_t (*)(int, int, int, int, int, int);
using FwdFn = int (*)(const void*, const void*, const void*, void*, float*, int, int, int, int, float, int, int, void*);
using FwdBwdFn = int (*)(const void*, const void*, const void*, const void*, void*, float*, void*, void*, void*, void*,
                         size_t, int, int, int, int, float, int, int, void*);
using BwdFn = int (*)(const void*, const void*, const void*, const void*, const float*, const void*, void*, void*, void*,
                      void*, size_t, int, int, int, int, float, int, int, void*);
using DecodeFn = int (*)(const void*, const void*, const void*, void*, void*, const int*, void*, float*, void*, size_t,
                         int, int, int, int, int, int, float, int, void*);

WsFn ws_bytes;
DecWsFn dec_ws_bytes;
FwdFn c_fwd;
FwdBwdFn c_fwd_bwd;
BwdFn c_bwd;
DecodeFn c_decode;
PyObject* raw_stream;   // device index -> the current stream's handle

PyObject* not_mine() { Py_RETURN_NOTIMPLEMENTED; }

// a dense, contiguous GPU tensor of exactly torch.Tensor
const at::Tensor* plain(PyObject* o) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.is_contiguous() || at::isTensorSubclassLike(t))
    return nullptr;
  return &t;
}
bool like(const at::Tensor* t, const at::Tensor& ref) {
  return t && t->scalar_type() == ref.scalar_type() && t->device() == ref.device() && t->sizes() == ref.sizes();
}
bool is(const at::Tensor* t, at::IntArrayRef sizes, at::ScalarType type, const at::Tensor& ref) {
  return t && t->scalar_type() == type && t->device() == ref.device() && t->sizes() == sizes;
}
int dtype_code(const at::Tensor& t) {
  return t.scalar_type() == at::kBFloat16 ? 0 : t.scalar_type() == at::kFloat ? 1 : -1;
}
bool fits_int(at::IntArrayRef sizes) {
  for (int64_t s : sizes)
    if (s > INT_MAX) return false;
  return true;
}
bool get_scale(PyObject* o, int64_t d, float& s) {
  if (o == Py_None) {
    s = (float)(1.0 / std::sqrt((double)d));
    return d > 0;
  }
  if (!PyFloat_CheckExact(o)) return false;
  s = (float)PyFloat_AS_DOUBLE(o);
  return true;
}
bool get_stream(const at::Tensor& t, void*& st) {
  PyObject* idx = PyLong_FromLong(t.get_device());
  if (!idx) return false;
  PyObject* r = PyObject_CallOneArg(raw_stream, idx);
  Py_DECREF(idx);
  if (!r) return false;
  st = PyLong_AsVoidPtr(r);
  Py_DECREF(r);
  return !PyErr_Occurred();
}
// the caller's workspace, or a new one of `need` bytes (at least one) in `own`
bool get_workspace(PyObject* o, size_t need, const at::Tensor& ref, at::Tensor& own, void*& p, size_t& bytes) {
  if (o == Py_None) {
    bytes = std::max<size_t>(need, 1);
    own = at::empty({(int64_t)bytes}, ref.options().dtype(at::kByte));
    p = own.data_ptr();
    return true;
  }
  const at::Tensor* t = plain(o);
  if (!t || t->device() != ref.device()) return false;
  bytes = t->nbytes();
  p = t->data_ptr();
  return bytes >= need;
}
// N outputs: the caller's tuple, or new tensors; output `l` is the float32 row
// vector (-1: none), the others are like `ref`
template <int N> struct Outputs {
  at::Tensor t[N];
  void* p[N];
  bool get(PyObject* o, const at::Tensor& ref, int l) {
    const auto rows = ref.sizes().slice(0, ref.dim() - 1);
    if (o == Py_None) {
      for (int i = 0; i < N; ++i) {
        t[i] = i == l ? at::empty(rows, ref.options().dtype(at::kFloat)) : at::empty_like(ref);
        p[i] = t[i].data_ptr();
      }
      return true;
    }
    if (!PyTuple_CheckExact(o) || PyTuple_GET_SIZE(o) != N) return false;
    for (int i = 0; i < N; ++i) {
      const at::Tensor* x = plain(PyTuple_GET_ITEM(o, i));
      if (!(i == l ? is(x, rows, at::kFloat, ref) : like(x, ref))) return false;
      p[i] = x->data_ptr();
    }
    return true;
  }
  PyObject* answer(PyObject* o) {
    if (o != Py_None) return Py_NewRef(o);
    PyObject* r = PyTuple_New(N);
    if (!r) return nullptr;
    for (int i = 0; i < N; ++i) {
      PyObject* x = THPVariable_Wrap(std::move(t[i]));
      if (!x) {
        Py_DECREF(r);
        return nullptr;
      }
      PyTuple_SET_ITEM(r, i, x);
    }
    return r;
  }
};
// C++ exceptions (a failed allocation) become the Python errors torch gives
template <typename F> PyObject* guarded(F f) {
  HANDLE_TH_ERRORS
  return f();
  END_HANDLE_TH_ERRORS
}
template <typename F> int released(F f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}

// fwd(q, k, v, scale, causal, out)
PyObject* fwd(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&]() -> PyObject* {
    if (na != 6) return not_mine();
    const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]);
    float scale;
    if (!q || q->dim() != 4 || !like(k, *q) || !like(v, *q) || !PyBool_Check(a[4]) || !fits_int(q->sizes()) ||
        dtype_code(*q) < 0 || !get_scale(a[3], q->size(3), scale))
      return not_mine();
    Outputs<2> out;
    if (!out.get(a[5], *q, 1)) return not_mine();
    void* st;
    if (!get_stream(*q, st)) return nullptr;
    const auto s = q->sizes();
    const int rc = released([&] {
      return c_fwd(q->data_ptr(), k->data_ptr(), v->data_ptr(), out.p[0], (float*)out.p[1], s[0], s[1], s[2], s[3], scale,
                   a[4] == Py_True, dtype_code(*q), st);
    });
    return rc ? PyLong_FromLong(rc) : out.answer(a[5]);
  });
}

// fwd_bwd(q, k, v, do, scale, causal, out, workspace)
PyObject* fwd_bwd(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&]() -> PyObject* {
    if (na != 8) return not_mine();
    const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]), *g = plain(a[3]);
    float scale;
    if (!q || q->dim() != 4 || !like(k, *q) || !like(v, *q) || !like(g, *q) || !PyBool_Check(a[5]) ||
        !fits_int(q->sizes()) || dtype_code(*q) < 0 || !get_scale(a[4], q->size(3), scale))
      return not_mine();
    const auto s = q->sizes();
    Outputs<5> out;
    at::Tensor own;
    void *ws, *st;
    size_t bytes;
    if (!out.get(a[6], *q, 1) || !get_workspace(a[7], ws_bytes(s[0], s[1], s[2], s[3]), *q, own, ws, bytes)) return not_mine();
    if (!get_stream(*q, st)) return nullptr;
    const int rc = released([&] {
      return c_fwd_bwd(q->data_ptr(), k->data_ptr(), v->data_ptr(), g->data_ptr(), out.p[0], (float*)out.p[1], out.p[2],
                       out.p[3], out.p[4], ws, bytes, s[0], s[1], s[2], s[3], scale, a[5] == Py_True, dtype_code(*q), st);
    });
    return rc ? PyLong_FromLong(rc) : out.answer(a[6]);
  });
}

// bwd(q, k, v, o, lse, do, scale, causal, out, workspace)
PyObject* bwd(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&]() -> PyObject* {
    if (na != 10) return not_mine();
    const at::Tensor *q = plain(a[0]), *k = plain(a[1]), *v = plain(a[2]), *o = plain(a[3]), *l = plain(a[4]), *g = plain(a[5]);
    float scale;
    if (!q || q->dim() != 4 || !like(k, *q) || !like(v, *q) || !like(o, *q) || !like(g, *q) ||
        !is(l, q->sizes().slice(0, 3), at::kFloat, *q) || !PyBool_Check(a[7]) || !fits_int(q->sizes()) ||
        dtype_code(*q) < 0 || !get_scale(a[6], q->size(3), scale))
      return not_mine();
    const auto s = q->sizes();
    Outputs<3> out;
    at::Tensor own;
    void *ws, *st;
    size_t bytes;
    if (!out.get(a[8], *q, -1) || !get_workspace(a[9], ws_bytes(s[0], s[1], s[2], s[3]), *q, own, ws, bytes)) return not_mine();
    if (!get_stream(*q, st)) return nullptr;
    const int rc = released([&] {
      return c_bwd(q->data_ptr(), k->data_ptr(), v->data_ptr(), o->data_ptr(), (const float*)l->data_ptr(), g->data_ptr(),
                   out.p[0], out.p[1], out.p[2], ws, bytes, s[0], s[1], s[2], s[3], scale, a[7] == Py_True, dtype_code(*q), st);
    });
    return rc ? PyLong_FromLong(rc) : out.answer(a[8]);
  });
}

// decode(q, k_cache, v_cache, k_new, v_new, cache_lens, n, scale, out, workspace)
PyObject* decode(PyObject*, PyObject* const* a, Py_ssize_t na) {
  return guarded([&]() -> PyObject* {
    if (na != 10) return not_mine();
    const at::Tensor *q = plain(a[0]), *kc = plain(a[1]), *vc = plain(a[2]), *kn = nullptr, *vn = nullptr, *lens = nullptr;
    float scale;
    if (!q || q->dim() != 3 || !kc || kc->dim() != 4 || !like(vc, *kc) || kc->scalar_type() != q->scalar_type() ||
        kc->device() != q->device() || kc->size(0) != q->size(0) || kc->size(3) != q->size(2) || !fits_int(q->sizes()) ||
        !fits_int(kc->sizes()) || dtype_code(*q) < 0 || !PyLong_CheckExact(a[6]) || !get_scale(a[7], q->size(2), scale))
      return not_mine();
    const int64_t B = q->size(0), Hq = q->size(1), d = q->size(2), Hkv = kc->size(1), n_cap = kc->size(2);
    if (a[3] != Py_None) {
      const int64_t rows[3] = {B, Hkv, d};
      kn = plain(a[3]), vn = plain(a[4]);
      if (!is(kn, rows, q->scalar_type(), *q) || !is(vn, rows, q->scalar_type(), *q)) return not_mine();
    }
    if (a[5] != Py_None) {
      lens = plain(a[5]);
      if (!is(lens, {B}, at::kInt, *q)) return not_mine();
    }
    int over;
    const long n = PyLong_AsLongAndOverflow(a[6], &over);
    if (over || n < INT_MIN || n > INT_MAX) return not_mine();
    if (n == -1 && PyErr_Occurred()) return nullptr;
    Outputs<2> out;
    if (!out.get(a[8], *q, 1)) return not_mine();
    const size_t need = dec_ws_bytes(B, Hq, Hkv, n, d, kn != nullptr);
    at::Tensor own;
    void *ws = nullptr, *st;
    size_t bytes = 0;
    if ((need > 0 || a[9] != Py_None) && !get_workspace(a[9], need, *q, own, ws, bytes)) return not_mine();
    if (!get_stream(*q, st)) return nullptr;
    const int rc = released([&] {
      return c_decode(q->data_ptr(), kn ? kn->data_ptr() : nullptr, vn ? vn->data_ptr() : nullptr, kc->data_ptr(),
                      vc->data_ptr(), lens ? (const int*)lens->data_ptr() : nullptr, out.p[0], (float*)out.p[1], ws, bytes,
                      B, Hq, Hkv, n, n_cap, d, scale, dtype_code(*q), st);
    });
    return rc ? PyLong_FromLong(rc) : out.answer(a[8]);
  });
}

// bind(workspace_bytes, decode_workspace_bytes, fwd, fwd_bwd, bwd, decode
//      [addresses], function that gives a device's current raw stream)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t na) {
  if (na != 7) {
    PyErr_SetString(PyExc_TypeError, "bind takes six addresses and a function");
    return nullptr;
  }
  void* p[6];
  for (int i = 0; i < 6; ++i) {
    p[i] = PyLong_AsVoidPtr(a[i]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "bind: null address");
      return nullptr;
    }
  }
  ws_bytes = (WsFn)p[0];
  dec_ws_bytes = (DecWsFn)p[1];
  c_fwd = (FwdFn)p[2];
  c_fwd_bwd = (FwdBwdFn)p[3];
  c_bwd = (BwdFn)p[4];
  c_decode = (DecodeFn)p[5];
  Py_XSETREF(raw_stream, Py_NewRef(a[6]));
  Py_RETURN_NONE;
}

#define FAST(f) reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(f)), METH_FASTCALL
PyMethodDef methods[] = {{"bind", FAST(bind), nullptr},       {"fwd", FAST(fwd), nullptr}, {"fwd_bwd", FAST(fwd_bwd), nullptr},
                         {"bwd", FAST(bwd), nullptr},         {"decode", FAST(decode), nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
