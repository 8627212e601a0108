// The calls of the Python binding for the arguments that they are made with in earnest: checks, extents and pointers in
// native code, then the entry point.  Host time is what bounds a small call: a lookup of two tables spent 7.9 us in Python
// attribute accesses around a kernel of 3.9.
//
// Every function returns the entry point's status, or -1 for whatever it does not know to be right -- a wrong type, dtype,
// shape or layout, a tensor subclass or wrapper, more than 8 layers or tables --, without having called anything: the binding
// then takes its general path, which decides and raises.  Nothing is kept between calls.
#include <torch/csrc/autograd/python_variable.h>

#include <c10/hip/HIPStream.h>

#include <cstdint>

namespace {

typedef int (*tbmm_t)(const float*, const float*, float*, int64_t, int64_t, int64_t, int64_t, void*);
typedef int (*tbmm_ws_t)(const float*, const float*, float*, int64_t, int64_t, int64_t, int64_t, void*, size_t, void*);
typedef int (*mlp_t)(const float*, int64_t, int32_t, const int64_t*, const float* const*, const float* const*, float* const*, void*, size_t, void*);
typedef int (*gconv_t)(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, void*);
typedef int (*kron_t)(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int64_t, int64_t, void*);
typedef int (*sconv_t)(const float*, const float*, const float*, float*, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                       void*);
typedef int (*lut_t)(int32_t, const float* const*, const int32_t* const*, float* const*, const int64_t*, const int64_t*, int64_t, int64_t, void*);

constexpr int kMost = 8;  // layers, tables

// A dense contiguous GPU tensor of `dims` dimensions, exactly torch's own (or a Parameter), behind no wrapper.
struct Arg {
  const int64_t* size = nullptr;
  void* data = nullptr;
};

bool take(PyObject* o, c10::ScalarType type, int64_t dims, Arg* a) {
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.scalar_type() != type || t.layout() != c10::kStrided) return false;
  const c10::TensorImpl* impl = t.unsafeGetTensorImpl();
  if (impl->has_symbolic_sizes_strides() || !impl->has_storage()) return false;
  using K = c10::DispatchKey;
  if (impl->key_set().has_any(c10::DispatchKeySet({K::FuncTorchBatched, K::FuncTorchGradWrapper, K::Functionalize, K::Python, K::Batched})))
    return false;
  if (t.dim() != dims || !t.is_contiguous()) return false;
  a->size = t.sizes().data();
  a->data = t.data_ptr();
  return true;
}
bool take(PyObject* o, int64_t dims, Arg* a) { return take(o, c10::kFloat, dims, a); }

bool stream_of(PyObject* o, void** s) {
  if (o == Py_None) {
    *s = c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  if (!PyLong_CheckExact(o)) return false;
  *s = PyLong_AsVoidPtr(o);
  if (!*s && PyErr_Occurred()) {
    PyErr_Clear();
    return false;
  }
  return true;
}

// Items of a list or tuple of n objects.
PyObject** items(PyObject* o, Py_ssize_t n) {
  if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) return nullptr;
  return PySequence_Fast_GET_SIZE(o) == n ? PySequence_Fast_ITEMS(o) : nullptr;
}

// An entry point from its address.
template <typename T>
bool entry_of(PyObject* o, T* entry) {
  if (!PyLong_CheckExact(o)) return false;
  *entry = reinterpret_cast<T>(PyLong_AsVoidPtr(o));
  return *entry || !PyErr_Occurred();
}

// Runs `body`, which returns a status or -1; what throws (a tensor without memory, for one) is left to the general path.
template <typename F>
PyObject* guarded(F body) {
  int st = -1;
  try {
    st = body();
  } catch (...) {
    st = -1;
  }
  if (PyErr_Occurred()) PyErr_Clear();
  return PyLong_FromLong(st);
}

// The call itself, without the interpreter's lock; its arguments are evaluated with it.
struct Unlocked {
  PyThreadState* const state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};
template <typename... P, typename... A>
int call(int (*entry)(P...), A... args) {
  Unlocked u;
  return entry(args...);
}

inline const float* f(const Arg& a) { return static_cast<const float*>(a.data); }
inline float* out(const Arg& a) { return static_cast<float*>(a.data); }

// (entry, X, Y, Z, stream)
PyObject* call_tbmm(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg X, Y, Z;
    void* s;
    if (n != 5 || !take(v[1], 3, &X) || !take(v[2], 3, &Y) || !take(v[3], 3, &Z) || !stream_of(v[4], &s)) return -1;
    const int64_t B = X.size[0], N = X.size[1], K = X.size[2], M = Y.size[1];
    if (Y.size[0] != B || Y.size[2] != K || Z.size[0] != B || Z.size[1] != N || Z.size[2] != M) return -1;
    tbmm_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(X), f(Y), out(Z), B, N, M, K, s);
  });
}

// (entry, X, Y, Z, workspace, stream)
PyObject* call_tbmm_ws(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg X, Y, Z, W;
    void* s;
    if (n != 6 || !take(v[1], 3, &X) || !take(v[2], 3, &Y) || !take(v[3], 3, &Z) || !take(v[4], c10::kByte, 1, &W) || !stream_of(v[5], &s)) return -1;
    const int64_t B = X.size[0], N = X.size[1], K = X.size[2], M = Y.size[1];
    if (Y.size[0] != B || Y.size[2] != K || Z.size[0] != B || Z.size[1] != N || Z.size[2] != M) return -1;
    tbmm_ws_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(X), f(Y), out(Z), B, N, M, K, W.data, (size_t)W.size[0], s);
  });
}

// (entry, I, W, bias, O, workspace or None, stream)
PyObject* call_mlp(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg I, ws;
    void* s;
    if (n != 7 || !take(v[1], 2, &I) || !(PyList_CheckExact(v[2]) || PyTuple_CheckExact(v[2]))) return -1;
    const Py_ssize_t layers = PySequence_Fast_GET_SIZE(v[2]);
    if (layers < 1 || layers > kMost) return -1;
    PyObject **W = items(v[2], layers), **b = items(v[3], layers), **O = items(v[4], layers);
    if (!W || !b || !O) return -1;
    const int64_t batch = I.size[0];
    int64_t dims[kMost + 1] = {I.size[1]};
    const float *Wp[kMost], *bp[kMost];
    float* Op[kMost];
    for (Py_ssize_t l = 0; l < layers; l++) {
      Arg w, c, o;
      if (!take(W[l], 2, &w) || !take(b[l], 1, &c) || w.size[1] != dims[l] || c.size[0] != w.size[0]) return -1;
      dims[l + 1] = w.size[0];
      if (O[l] != Py_None && (!take(O[l], 2, &o) || o.size[0] != batch || o.size[1] != dims[l + 1])) return -1;
      Wp[l] = f(w);
      bp[l] = f(c);
      Op[l] = out(o);
    }
    if ((v[5] != Py_None && !take(v[5], c10::kByte, 1, &ws)) || !stream_of(v[6], &s)) return -1;
    const size_t bytes = ws.size ? (size_t)ws.size[0] : 0;
    mlp_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(I), batch, (int32_t)layers, dims, Wp, bp, Op, ws.data, bytes, s);
  });
}

// (entry, I, W1, bias or None, O, stream)
PyObject* call_gconv(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg I, W, b, O;
    void* s;
    if (n != 6 || !take(v[1], 5, &I) || !take(v[2], 5, &W) || (v[3] != Py_None && !take(v[3], 1, &b)) || !take(v[4], 5, &O) || !stream_of(v[5], &s))
      return -1;
    const int64_t N = I.size[0], G = I.size[1], C = I.size[2], H = I.size[3], Wd = I.size[4], F = W.size[1], KH = W.size[3], KW = W.size[4];
    if (W.size[0] != G || W.size[2] != C || (b.size && b.size[0] != G * F)) return -1;
    if (O.size[0] != N || O.size[1] != G || O.size[2] != F || O.size[3] != H - KH + 1 || O.size[4] != Wd - KW + 1) return -1;
    gconv_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(I), f(W), f(b), out(O), N, G, C, F, H, Wd, KH, KW, s);
  });
}

// (entry, W1, W2, X, Y, stream)
PyObject* call_kron(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg W1, W2, X, Y;
    void* s;
    if (n != 6 || !take(v[1], 2, &W1) || !take(v[2], 2, &W2) || !take(v[3], 3, &X) || !take(v[4], 3, &Y) || !stream_of(v[5], &s)) return -1;
    const int64_t I = W1.size[0], K = W1.size[1], J = W2.size[0], L = W2.size[1], B = X.size[0];
    if (X.size[1] != K || X.size[2] != L || Y.size[0] != B || Y.size[1] != I || Y.size[2] != J) return -1;
    kron_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(W1), f(W2), f(X), out(Y), B, I, K, J, L, s);
  });
}

// (entry, I, Wt, bias or None, O, sh, sw, stream)
PyObject* call_sconv(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    Arg I, W, b, O;
    void* s;
    if (n != 8 || !take(v[1], 4, &I) || !take(v[2], 4, &W) || (v[3] != Py_None && !take(v[3], 1, &b)) || !take(v[4], 4, &O) || !stream_of(v[7], &s))
      return -1;
    if (!PyLong_CheckExact(v[5]) || !PyLong_CheckExact(v[6])) return -1;
    const int64_t sh = PyLong_AsLongLong(v[5]), sw = PyLong_AsLongLong(v[6]);
    const int64_t N = I.size[0], C = I.size[1], H = I.size[2], Wd = I.size[3], F = W.size[0], KH = W.size[2], KW = W.size[3];
    if (W.size[1] != C || (b.size && b.size[0] != F) || sh < 1 || sw < 1 || KH < 1 || KH > H || KW < 1 || KW > Wd) return -1;
    if (O.size[0] != N || O.size[1] != F || O.size[2] != (H - KH) / sh + 1 || O.size[3] != (Wd - KW) / sw + 1) return -1;
    sconv_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, f(I), f(W), f(b), out(O), N, C, F, H, Wd, KH, KW, sh, sw, s);
  });
}

// (entry, LUT, Idx, O, stream)
PyObject* call_lut(PyObject*, PyObject* const* v, Py_ssize_t n) {
  return guarded([&]() -> int {
    void* s;
    if (n != 5 || !(PyList_CheckExact(v[1]) || PyTuple_CheckExact(v[1]))) return -1;
    const Py_ssize_t tables = PySequence_Fast_GET_SIZE(v[1]);
    if (tables < 1 || tables > kMost) return -1;
    PyObject **T = items(v[1], tables), **X = items(v[2], tables), **O = items(v[3], tables);
    if (!T || !X || !O) return -1;
    const float* Tp[kMost];
    const int32_t* Xp[kMost];
    float* Op[kMost];
    int64_t E[kMost], L[kMost], B = 0, D = 0;
    for (Py_ssize_t t = 0; t < tables; t++) {
      Arg a, x, o;
      if (!take(T[t], 2, &a) || !take(X[t], c10::kInt, 2, &x) || !take(O[t], 2, &o)) return -1;
      if (t == 0) {
        B = o.size[0];
        D = o.size[1];
      }
      if (o.size[0] != B || o.size[1] != D || a.size[1] != D || x.size[0] != B) return -1;
      Tp[t] = f(a);
      Xp[t] = static_cast<const int32_t*>(x.data);
      Op[t] = out(o);
      E[t] = a.size[0];
      L[t] = x.size[1];
    }
    if (!stream_of(v[4], &s)) return -1;
    lut_t entry;
    if (!entry_of(v[0], &entry)) return -1;
    return call(entry, (int32_t)tables, Tp, Xp, Op, E, L, D, B, s);
  });
}

template <PyObject* (*F)(PyObject*, PyObject* const*, Py_ssize_t)>
PyMethodDef method(const char* name) {
  return {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(F)), METH_FASTCALL, nullptr};
}

PyMethodDef methods[] = {method<call_tbmm>("tbmm"),   method<call_tbmm_ws>("tbmm_ws"), method<call_mlp>("mlp"),
                         method<call_gconv>("gconv"), method<call_kron>("kron"),       method<call_sconv>("sconv"),
                         method<call_lut>("lut"),     {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_fast", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fast(void) { return PyModule_Create(&module); }
