// Python entry of the calls that a layer makes on every step (module _pit_native): takes the tensors as they are, reads sizes,
// strides, types and addresses, and calls the library.  Marshalling the same arguments through ctypes costs 2.6 - 3.3 us per call,
// as much as a kernel launch or two; by this module a call is 0.4 us, 0.15 of it here.
//
// A function returns the library's status, or None for arguments out of the ordinary (a subclass of Tensor, a type without a
// code, a tensor of other dimensions, a number that is not a Python int or does not fit its C type): pit.py then takes its
// general path, which accepts or refuses them as it always has.  Nothing is kept from one call to the next.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>
#include <algorithm>
#include <climits>
#include <vector>
#include "../../include/pit.h"

namespace {

using at::Tensor;

bool is_tensor(PyObject* o) { return THPVariable_CheckExact(o); }
const Tensor& tensor(PyObject* o) { return THPVariable_Unpack(o); }

// One call's arguments; `ok` turns false at the first that is out of the ordinary.
struct Args {
  PyObject* const* a;
  bool ok = true;
  const Tensor* t(int i) {
    if (!is_tensor(a[i])) { ok = false; return nullptr; }
    return &tensor(a[i]);
  }
  void* ptr(int i, bool none_allowed = false) {
    if (none_allowed && a[i] == Py_None) return nullptr;
    const Tensor* x = t(i);
    return x ? x->data_ptr() : nullptr;
  }
  long long integer(int i) {
    if (!PyLong_Check(a[i])) { ok = false; return 0; }
    int over = 0;
    const long long v = PyLong_AsLongLongAndOverflow(a[i], &over);
    if (over != 0) { ok = false; return 0; }
    return v;
  }
  int i32(int i) {
    const long long v = integer(i);
    if (v < INT_MIN || v > INT_MAX) { ok = false; return 0; }
    return (int)v;
  }
  void* stream(int i) { return reinterpret_cast<void*>(static_cast<intptr_t>(integer(i))); }
  int code(const Tensor* x) {
    if (x == nullptr) return -1;
    switch (x->scalar_type()) {
      case at::kByte: case at::kBool: return PIT_U8;
      case at::kHalf: return PIT_F16;
      case at::kBFloat16: return PIT_BF16;
      case at::kFloat: return PIT_F32;
      default: ok = false; return -1;
    }
  }
  // a matrix whose rows are contiguous (an empty one may have any strides where `empty_any`)
  bool matrix(const Tensor* x, bool empty_any = false) {
    if (x == nullptr || x->dim() != 2 || (x->stride(1) != 1 && !(empty_any && x->numel() == 0))) { ok = false; return false; }
    return true;
  }
  bool size32(const Tensor& x) {
    for (int d = 0; d < x.dim(); ++d)
      if (x.size(d) > INT_MAX) { ok = false; return false; }
    return true;
  }
};

// row pitch of a matrix; of a single row, whose stride says nothing, at least its length
int64_t pitch(const Tensor& x) { return x.size(0) > 1 ? x.stride(0) : std::max<int64_t>(x.size(1), x.stride(0)); }

template <typename F> int unlocked(F&& f) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = f();
  Py_END_ALLOW_THREADS
  return rc;
}
// f(args) -> status; anything out of the ordinary, a C++ exception included (a tensor without storage), is None
template <typename F> PyObject* guarded(PyObject* const* args, Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) { PyErr_SetString(PyExc_TypeError, "_pit_native: number of arguments"); return nullptr; }
  int rc = 0;
  bool ok = false;
  try {
    Args a{args};
    ok = f(a, rc);
  } catch (const std::exception&) {
    ok = false;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  if (!ok) Py_RETURN_NONE;
  return PyLong_FromLong(rc);
}
// seg_ptr, idx, bits (or None), nseg, cap from argument i on
pit_index index_of(Args& a, int i) {
  pit_index ix;
  ix.seg_ptr = static_cast<int32_t*>(a.ptr(i));
  ix.idx = static_cast<int32_t*>(a.ptr(i + 1));
  ix.bits = static_cast<uint32_t*>(a.ptr(i + 2, true));
  ix.nseg = a.i32(i + 3);
  ix.cap = a.i32(i + 4);
  return ix;
}

// src, mt_rows, mt_cols, pit_dim, seg_ptr, idx, bits, nseg, cap, ws, stream
PyObject* build_index(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 11, [](Args& a, int& rc) {
    const Tensor* src = a.t(0);
    if (!a.matrix(src) || !a.size32(*src)) return false;
    const int dt = a.code(src), mr = a.i32(1), mc = a.i32(2), pd = a.i32(3);
    pit_index ix = index_of(a, 4);
    void* ws = a.ptr(9);
    void* st = a.stream(10);
    const void* p = src->data_ptr();
    if (!a.ok) return false;
    const size_t bytes = (size_t)a.t(9)->numel();
    const int rows = (int)src->size(0), cols = (int)src->size(1);
    const int64_t ld = pitch(*src);
    rc = unlocked([&] { return pit_build_index(p, dt, rows, cols, ld, mr, mc, pd, &ix, ws, bytes, st); });
    return true;
  });
}

// H, out_xt, seg_ptr, idx, bits, nseg, cap, ws, stream
PyObject* relu_channel_major_index(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 9, [](Args& a, int& rc) {
    const Tensor *H = a.t(0), *X = a.t(1);
    if (!a.matrix(H) || !a.size32(*H) || X == nullptr || X->dim() < 1) return false;
    const int dt = a.code(H);
    pit_index ix = index_of(a, 2);
    void* ws = a.ptr(7);
    void* st = a.stream(8);
    const void* h = H->data_ptr();
    void* x = X->data_ptr();
    if (!a.ok) return false;
    const size_t bytes = (size_t)a.t(7)->numel();
    const int tokens = (int)H->size(0), channels = (int)H->size(1);
    const int64_t ldh = pitch(*H), ldx = channels > 1 ? X->stride(0) : std::max<int64_t>(tokens, X->stride(0));
    rc = unlocked([&] { return pit_relu_channel_major_index(h, ldh, tokens, channels, dt, x, ldx, &ix, ws, bytes, st); });
    return true;
  });
}

// mode, A, B, seg_ptr (None: no index), idx, bits, nseg, cap, mt, M, N, K, out, zero_uncovered, stream
PyObject* sread_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 15, [](Args& a, int& rc) {
    const Tensor *A = a.t(1), *B = a.t(2), *C = a.t(12);
    if (!a.matrix(A, true) || !a.matrix(B, true) || C == nullptr || C->dim() < 1 || A->scalar_type() != B->scalar_type()) return false;
    const int mode = a.i32(0), dt = a.code(B), cdt = a.code(C), mt = a.i32(8), M = a.i32(9), N = a.i32(10), K = a.i32(11), z = a.i32(13);
    const bool with = a.a[3] != Py_None;
    pit_index ix = {};
    if (with) ix = index_of(a, 3);
    void* st = a.stream(14);
    const void *pa = A->data_ptr(), *pb = B->data_ptr();
    void* pc = C->data_ptr();
    if (!a.ok) return false;
    const int64_t lda = A->stride(0), ldb = B->stride(0), ldc = C->stride(0);
    rc = unlocked([&] { return pit_sread_gemm(mode, pa, lda, pb, ldb, pc, ldc, M, N, K, dt, cdt, with ? &ix : nullptr, mt, z, st); });
    return true;
  });
}

// candidates (list of dicts), num_tiles, grid_tiles (lists of lists of ints), At, B, M, N, K, out, ws, stream -> (status, chosen)
PyObject* select_and_run_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  int chosen = -1;
  PyObject* rc = guarded(args, n, 11, [&](Args& a, int& status) {
    if (!PyList_CheckExact(a.a[0]) || !PyList_CheckExact(a.a[1]) || !PyList_CheckExact(a.a[2])) return false;
    const Py_ssize_t nc = PyList_GET_SIZE(a.a[0]), ns = PyList_GET_SIZE(a.a[1]);
    if (nc > 1024 || ns > 1024 || PyList_GET_SIZE(a.a[2]) != ns) return false;
    const auto integer = [](PyObject* o, int64_t& v) {     // (missing: the caller's default stays)
      if (o == nullptr) return true;
      int over = 0;
      if (!PyLong_Check(o)) return false;
      v = PyLong_AsLongLongAndOverflow(o, &over);
      return over == 0;
    };
    const auto real = [](PyObject* o, double& v) {
      if (o == nullptr) return true;
      if (!PyFloat_CheckExact(o)) return false;
      v = PyFloat_AS_DOUBLE(o);
      return true;
    };
    std::vector<pit_kernel_candidate> cand((size_t)nc);
    for (Py_ssize_t j = 0; j < nc; ++j) {
      PyObject* d = PyList_GET_ITEM(a.a[0], j);
      if (!PyDict_CheckExact(d)) return false;
      PyObject *r = PyDict_GetItemString(d, "mt_rows"), *c = PyDict_GetItemString(d, "mt_cols"), *t = PyDict_GetItemString(d, "tile_cost");
      int64_t mr = 0, mc = 0, dense = 0;
      double tile = 0.0, fixed = 0.0;
      if (!r || !c || !t || !integer(r, mr) || !integer(c, mc) || !integer(PyDict_GetItemString(d, "dense"), dense) || !real(t, tile) ||
          !real(PyDict_GetItemString(d, "fixed_cost"), fixed) || mr < INT_MIN || mr > INT_MAX || mc < INT_MIN || mc > INT_MAX) return false;
      pit_kernel_candidate k = {};
      k.mt_rows = (int32_t)mr; k.mt_cols = (int32_t)mc; k.dense = dense != 0; k.tile_cost = tile; k.fixed_cost = fixed;
      cand[(size_t)j] = k;
    }
    std::vector<int64_t> counts[2];
    for (int w = 0; w < 2; ++w)
      for (Py_ssize_t i = 0; i < ns; ++i) {
        PyObject* row = PyList_GET_ITEM(a.a[1 + w], i);
        if (!PyList_CheckExact(row) || PyList_GET_SIZE(row) != nc) return false;
        for (Py_ssize_t j = 0; j < nc; ++j) {
          int64_t v = 0;
          if (!integer(PyList_GET_ITEM(row, j), v)) return false;
          counts[w].push_back(v);
        }
      }
    for (auto& c : counts) c.resize(std::max<size_t>(c.size(), 1));        // (an address even without samples)
    cand.resize(std::max<size_t>(cand.size(), 1));
    const Tensor *A = a.t(3), *B = a.t(4), *C = a.t(8);
    if (!a.matrix(A, true) || !a.matrix(B, true) || C == nullptr || C->dim() < 1 || A->scalar_type() != B->scalar_type()) return false;
    const int dt = a.code(B), cdt = a.code(C), M = a.i32(5), N = a.i32(6), K = a.i32(7);
    void* ws = a.ptr(9);
    void* st = a.stream(10);
    const void *pa = A->data_ptr(), *pb = B->data_ptr();
    void* pc = C->data_ptr();
    if (!a.ok) return false;
    const size_t bytes = (size_t)a.t(9)->numel();
    const int64_t lda = A->stride(0), ldb = B->stride(0), ldc = C->stride(0);
    status = unlocked([&] {
      return pit_select_and_run_gemm(cand.data(), (int)nc, counts[0].data(), counts[1].data(), (int)ns, pa, lda, pb, ldb, pc, ldc, M, N, K, dt, cdt,
                                     ws, bytes, &chosen, st);
    });
    return true;
  });
  if (rc == nullptr || rc == Py_None) return rc;
  return Py_BuildValue("(Ni)", rc, chosen);
}

// X, expert_id, gate, W1, W2, out, act, status, ws, stream
PyObject* moe_dispatch_gemm(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 10, [](Args& a, int& rc) {
    const Tensor *X = a.t(0), *e = a.t(1), *W1 = a.t(3), *W2 = a.t(4), *Y = a.t(5);
    const Tensor* gate = a.a[2] == Py_None ? nullptr : a.t(2);
    if (!a.ok || X->dim() != 2 || W1->dim() != 3 || W2->dim() != 3) return false;
    const int64_t T = X->size(0), d = X->size(1), E = W1->size(0), f = W1->size(2);
    const bool regular = X->scalar_type() == W1->scalar_type() && X->scalar_type() == W2->scalar_type() && X->is_contiguous() &&
                         W1->is_contiguous() && W2->is_contiguous() && e->scalar_type() == at::kInt && e->is_contiguous() &&
                         W2->size(0) == E && W2->size(1) == f && W2->size(2) == d &&
                         (gate == nullptr || (gate->scalar_type() == at::kFloat && gate->is_contiguous()));
    if (!regular || !a.size32(*X) || !a.size32(*W1)) return false;
    const int dt = a.code(X), ydt = a.code(Y), act = a.i32(6);
    int32_t* status = static_cast<int32_t*>(a.ptr(7, true));
    void* ws = a.ptr(8);
    void* st = a.stream(9);
    const void *px = X->data_ptr(), *p1 = W1->data_ptr(), *p2 = W2->data_ptr();
    const int32_t* pe = static_cast<const int32_t*>(e->data_ptr());
    const float* pg = gate ? static_cast<const float*>(gate->data_ptr()) : nullptr;
    void* py = Y->data_ptr();
    if (!a.ok) return false;
    const size_t bytes = (size_t)a.t(8)->numel();
    rc = unlocked([&] { return pit_moe_dispatch_gemm(px, pe, pg, p1, p2, py, ydt, (int)T, (int)d, (int)f, (int)E, dt, act, status, ws, bytes, st); });
    return true;
  });
}

// Q, K, V, mask, scale, out, ws, stream
PyObject* sparse_attn(PyObject*, PyObject* const* args, Py_ssize_t n) {
  return guarded(args, n, 8, [](Args& a, int& rc) {
    const Tensor *Q = a.t(0), *K = a.t(1), *V = a.t(2), *m = a.t(3), *O = a.t(5);
    if (!a.ok || Q->dim() != 3 || !PyFloat_CheckExact(a.a[4])) return false;
    const bool regular = Q->scalar_type() == K->scalar_type() && Q->scalar_type() == V->scalar_type() && Q->is_contiguous() &&
                         K->is_contiguous() && V->is_contiguous() && K->sizes() == Q->sizes() && V->sizes() == Q->sizes() &&
                         (m->scalar_type() == at::kByte || m->scalar_type() == at::kBool) && m->is_contiguous() && m->dim() == 2 &&
                         m->size(0) == Q->size(1) && m->size(1) == Q->size(1);
    if (!regular || !a.size32(*Q)) return false;
    const int dt = a.code(Q), odt = a.code(O);
    const float scale = (float)PyFloat_AS_DOUBLE(a.a[4]);
    void* ws = a.ptr(6);
    void* st = a.stream(7);
    const void *pq = Q->data_ptr(), *pk = K->data_ptr(), *pv = V->data_ptr(), *pm = m->data_ptr();
    void* po = O->data_ptr();
    if (!a.ok) return false;
    const size_t bytes = (size_t)a.t(6)->numel();
    const int H = (int)Q->size(0), S = (int)Q->size(1), D = (int)Q->size(2);
    rc = unlocked([&] { return pit_sparse_attn(pq, pk, pv, static_cast<const uint8_t*>(pm), po, odt, H, S, D, scale, dt, ws, bytes, st); });
    return true;
  });
}

PyMethodDef methods[] = {
    {"build_index", (PyCFunction)(void (*)(void))build_index, METH_FASTCALL, nullptr},
    {"relu_channel_major_index", (PyCFunction)(void (*)(void))relu_channel_major_index, METH_FASTCALL, nullptr},
    {"sread_gemm", (PyCFunction)(void (*)(void))sread_gemm, METH_FASTCALL, nullptr},
    {"select_and_run_gemm", (PyCFunction)(void (*)(void))select_and_run_gemm, METH_FASTCALL, nullptr},
    {"moe_dispatch_gemm", (PyCFunction)(void (*)(void))moe_dispatch_gemm, METH_FASTCALL, nullptr},
    {"sparse_attn", (PyCFunction)(void (*)(void))sparse_attn, METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pit_native", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pit_native(void) { return PyModule_Create(&module); }
