// The common form of the binding's calls in native code: plain contiguous tensors on the
// current device, outputs allocated here, the current stream. A call of this form costs
// the host two or three microseconds beside its kernel launch, against six to eight for
// the same steps in Python (checks, allocations, argument conversion), which is what the
// smallest calls were bound by. Every function returns None for anything else (another
// type, device, layout or shape), and binding.py then takes its own path with its own
// errors; a status other than 0 comes back as an int.
//
// Nothing is kept between calls but the addresses of the library's functions and of
// torch's accessor of the current stream's raw handle.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/core/impl/VirtualGuardImpl.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

PyObject* g_raw_stream = nullptr;   // torch._C._cuda_getCurrentRawStream
enum { kFp32 = 0, kBf16 = 1 };

// A plain dense tensor in GPU memory with storage of its own type; no subclass.
bool plain(PyObject* o, at::Tensor& t) {
  if (!THPVariable_CheckExact(o)) return false;
  t = THPVariable_Unpack(o);
  return t.defined() && t.device().type() == c10::DeviceType::CUDA && t.layout() == c10::kStrided &&
         t.has_storage() && t.is_contiguous();
}
int dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return kFp32;
  if (t.scalar_type() == at::kBFloat16) return kBf16;
  return -1;
}
bool on_current_device(const at::Tensor& t) {
  return c10::impl::VirtualGuardImpl(c10::DeviceType::CUDA).getDevice() == t.device();
}
bool same(const at::Tensor& a, const at::Tensor& b) {
  return a.scalar_type() == b.scalar_type() && a.numel() == b.numel() && a.device() == b.device();
}
// The current stream's raw handle; false with a Python error set.
bool stream_of(const at::Tensor& t, void*& s) {
  PyObject* index = PyLong_FromLong(t.device().index());
  if (index == nullptr) return false;
  PyObject* handle = PyObject_CallOneArg(g_raw_stream, index);
  Py_DECREF(index);
  if (handle == nullptr) return false;
  s = PyLong_AsVoidPtr(handle);
  Py_DECREF(handle);
  return !PyErr_Occurred();
}
at::Tensor words(int64_t count, const at::Tensor& like) {
  return at::empty({count}, like.options().dtype(at::kInt));
}
int64_t code_words(int64_t n) { return (n + 15) / 16; }

template <class... T>
PyObject* result(int status, const T&... t) {
  if (status != 0) return PyLong_FromLong(status);
  if constexpr (sizeof...(T) == 1) {
    return THPVariable_Wrap((t, ...));
  } else {
    PyObject* out = PyTuple_New(sizeof...(T));
    if (out == nullptr) return nullptr;
    Py_ssize_t i = 0;
    bool ok = true;
    auto add = [&](const at::Tensor& v) {
      PyObject* o = ok ? THPVariable_Wrap(v) : nullptr;
      if (o == nullptr) ok = false;
      else PyTuple_SET_ITEM(out, i++, o);
    };
    (add(t), ...);
    if (ok) return out;
    Py_DECREF(out);
    return nullptr;
  }
}

// Allocations and launches run without the interpreter's lock, as torch's and ctypes' do.
struct NoGil {
  PyThreadState* state = PyEval_SaveThread();
  ~NoGil() { PyEval_RestoreThread(state); }
};

template <class F>
F address(PyObject* o) {
  return reinterpret_cast<F>(PyLong_AsVoidPtr(o));
}

// (function, x) -> (y, codes)
PyObject* act_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x;
  if (n != 2 || !plain(a[1], x)) Py_RETURN_NONE;
  const int dt = dtype_of(x);
  if (dt < 0 || !on_current_device(x)) Py_RETURN_NONE;
  void* s;
  if (!stream_of(x, s)) return nullptr;
  at::Tensor y, codes;
  const auto f = address<int (*)(int, int64_t, const void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    y = at::empty_like(x);
    codes = words(code_words(x.numel()), x);
    status = f(dt, x.numel(), x.data_ptr(), y.data_ptr(), codes.data_ptr(), s);
  }
  return result(status, y, codes);
  END_HANDLE_TH_ERRORS
}

// (function, dy, codes) -> dx
PyObject* act_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor dy, codes;
  if (n != 3 || !plain(a[1], dy) || !plain(a[2], codes)) Py_RETURN_NONE;
  const int dt = dtype_of(dy);
  if (dt < 0 || !on_current_device(dy) || codes.device() != dy.device() || codes.scalar_type() != at::kInt ||
      codes.numel() < code_words(dy.numel()))
    Py_RETURN_NONE;
  void* s;
  if (!stream_of(dy, s)) return nullptr;
  at::Tensor dx;
  const auto f = address<int (*)(int, int64_t, const void*, const void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    dx = at::empty_like(dy);
    status = f(dt, dy.numel(), dy.data_ptr(), codes.data_ptr(), dx.data_ptr(), s);
  }
  return result(status, dx);
  END_HANDLE_TH_ERRORS
}

// (function, g, u) -> (h, s, codes)
PyObject* glu_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor g, u;
  if (n != 3 || !plain(a[1], g) || !plain(a[2], u)) Py_RETURN_NONE;
  const int dt = dtype_of(g);
  if (dt < 0 || !on_current_device(g) || !same(u, g)) Py_RETURN_NONE;
  void* st;
  if (!stream_of(g, st)) return nullptr;
  at::Tensor h, s, codes;
  const auto f = address<int (*)(int, int64_t, const void*, const void*, void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    h = at::empty_like(g);
    s = at::empty_like(g);
    codes = words(code_words(g.numel()), g);
    status = f(dt, g.numel(), g.data_ptr(), u.data_ptr(), h.data_ptr(), s.data_ptr(), codes.data_ptr(), st);
  }
  return result(status, h, s, codes);
  END_HANDLE_TH_ERRORS
}

// (function, dh, u, s, codes) -> (dg, du)
PyObject* glu_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor dh, u, s, codes;
  if (n != 5 || !plain(a[1], dh) || !plain(a[2], u) || !plain(a[3], s) || !plain(a[4], codes)) Py_RETURN_NONE;
  const int dt = dtype_of(dh);
  if (dt < 0 || !on_current_device(dh) || !same(u, dh) || !same(s, dh) || codes.device() != dh.device() ||
      codes.scalar_type() != at::kInt || codes.numel() < code_words(dh.numel()))
    Py_RETURN_NONE;
  void* st;
  if (!stream_of(dh, st)) return nullptr;
  at::Tensor dg, du;
  const auto f = address<int (*)(int, int64_t, const void*, const void*, const void*, const void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    dg = at::empty_like(dh);
    du = at::empty_like(dh);
    status = f(dt, dh.numel(), dh.data_ptr(), u.data_ptr(), s.data_ptr(), codes.data_ptr(), dg.data_ptr(),
               du.data_ptr(), st);
  }
  return result(status, dg, du);
  END_HANDLE_TH_ERRORS
}

// (function, x, eps) -> (z, rstd)
PyObject* norm_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x;
  if (n != 3 || !PyFloat_CheckExact(a[2]) || !plain(a[1], x)) Py_RETURN_NONE;
  const int dt = dtype_of(x);
  if (dt < 0 || x.dim() == 0 || !on_current_device(x)) Py_RETURN_NONE;
  const int64_t cols = x.size(-1), rows = cols != 0 ? x.numel() / cols : 0;
  void* s;
  if (!stream_of(x, s)) return nullptr;
  at::Tensor z, rstd;
  const auto f = address<int (*)(int, int64_t, int64_t, float, const void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    z = at::empty_like(x);
    rstd = at::empty(x.sizes().slice(0, size_t(x.dim() - 1)), x.options().dtype(at::kFloat));
    status = f(dt, rows, cols, float(PyFloat_AS_DOUBLE(a[2])), x.data_ptr(), z.data_ptr(), rstd.data_ptr(), s);
  }
  return result(status, z, rstd);
  END_HANDLE_TH_ERRORS
}

// (function, dz, z, rstd) -> dx
PyObject* norm_bwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor dz, z, rstd;
  if (n != 4 || !plain(a[1], dz) || !plain(a[2], z) || !plain(a[3], rstd)) Py_RETURN_NONE;
  const int dt = dtype_of(dz);
  if (dt < 0 || dz.dim() == 0 || !on_current_device(dz) || !same(z, dz) || z.sizes() != dz.sizes()) Py_RETURN_NONE;
  const int64_t cols = dz.size(-1), rows = cols != 0 ? dz.numel() / cols : 0;
  if (rstd.device() != dz.device() || rstd.scalar_type() != at::kFloat || rstd.numel() != rows) Py_RETURN_NONE;
  void* s;
  if (!stream_of(dz, s)) return nullptr;
  at::Tensor dx;
  const auto f = address<int (*)(int, int64_t, int64_t, const void*, const void*, const void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    dx = at::empty_like(dz);
    status = f(dt, rows, cols, dz.data_ptr(), z.data_ptr(), rstd.data_ptr(), dx.data_ptr(), s);
  }
  return result(status, dx);
  END_HANDLE_TH_ERRORS
}

// Sizes of a layer: x [.., k] and w [n, k], both bf16; false if they are anything else.
bool layer(const at::Tensor& x, const at::Tensor& w, int64_t& m, c10::SmallVector<int64_t, 6>& out) {
  if (x.scalar_type() != at::kBFloat16 || w.scalar_type() != at::kBFloat16 || w.dim() != 2 || x.dim() == 0 ||
      x.size(-1) != w.size(1) || w.device() != x.device() || !on_current_device(x))
    return false;
  out.assign(x.sizes().begin(), x.sizes().end());
  out.back() = w.size(0);
  m = 1;
  for (size_t i = 0; i + 1 < out.size(); ++i) m *= out[i];
  return true;
}

// (function, activation, x, w, bias or None) -> (y, codes)
PyObject* linear_act_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x, w, b;
  int64_t m;
  c10::SmallVector<int64_t, 6> shape;
  if (n != 5 || !plain(a[2], x) || !plain(a[3], w) || !layer(x, w, m, shape)) Py_RETURN_NONE;
  if (a[4] != Py_None && (!plain(a[4], b) || b.scalar_type() != at::kBFloat16 || b.numel() != w.size(0) ||
                          b.device() != x.device()))
    Py_RETURN_NONE;
  void* s;
  if (!stream_of(x, s)) return nullptr;
  const int act = int(PyLong_AsLong(a[1]));
  at::Tensor y, codes;
  const auto f = address<int (*)(int, int, int64_t, int64_t, int64_t, const void*, const void*, const void*, void*,
                                 void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    y = at::empty(shape, x.options());
    codes = words(code_words(m * w.size(0)), x);
    status = f(act, kBf16, m, w.size(0), w.size(1), x.data_ptr(), w.data_ptr(),
               b.defined() ? b.data_ptr() : nullptr, y.data_ptr(), codes.data_ptr(), nullptr, s);
  }
  return result(status, y, codes);
  END_HANDLE_TH_ERRORS
}

// (function, x, w_gate, w_up) -> (h, s, u, codes)
PyObject* linear_swiglu_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x, wg, wu;
  int64_t m;
  c10::SmallVector<int64_t, 6> shape;
  if (n != 4 || !plain(a[1], x) || !plain(a[2], wg) || !plain(a[3], wu) || !layer(x, wg, m, shape) || !same(wu, wg) ||
      wu.sizes() != wg.sizes())
    Py_RETURN_NONE;
  void* st;
  if (!stream_of(x, st)) return nullptr;
  at::Tensor h, s, u, codes;
  const auto f = address<int (*)(int, int64_t, int64_t, int64_t, const void*, const void*, const void*, void*, void*,
                                 void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    h = at::empty(shape, x.options());
    s = at::empty(shape, x.options());
    u = at::empty(shape, x.options());
    codes = words(code_words(m * wg.size(0)), x);
    status = f(kBf16, m, wg.size(0), wg.size(1), x.data_ptr(), wg.data_ptr(), wu.data_ptr(), h.data_ptr(),
                s.data_ptr(), u.data_ptr(), codes.data_ptr(), nullptr, st);
  }
  return result(status, h, s, u, codes);
  END_HANDLE_TH_ERRORS
}

// (function, activation, x, w, eps, bias or None) -> (y, codes, z, rstd)
PyObject* norm_linear_act_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x, w, b;
  int64_t m;
  c10::SmallVector<int64_t, 6> shape;
  if (n != 6 || !PyFloat_CheckExact(a[4]) || !plain(a[2], x) || !plain(a[3], w) || !layer(x, w, m, shape))
    Py_RETURN_NONE;
  if (a[5] != Py_None && (!plain(a[5], b) || b.scalar_type() != at::kBFloat16 || b.numel() != w.size(0) ||
                          b.device() != x.device()))
    Py_RETURN_NONE;
  void* s;
  if (!stream_of(x, s)) return nullptr;
  const int act = int(PyLong_AsLong(a[1]));
  at::Tensor y, codes, z, rstd;
  const auto f = address<int (*)(int, int, int64_t, int64_t, int64_t, float, const void*, const void*, const void*,
                                 void*, void*, void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    y = at::empty(shape, x.options());
    z = at::empty(x.sizes(), x.options());
    rstd = at::empty({m}, x.options().dtype(at::kFloat));
    codes = words(code_words(m * w.size(0)), x);
    status = f(act, kBf16, m, w.size(0), w.size(1), float(PyFloat_AS_DOUBLE(a[4])), x.data_ptr(), w.data_ptr(),
               b.defined() ? b.data_ptr() : nullptr, y.data_ptr(), codes.data_ptr(), nullptr, z.data_ptr(),
               rstd.data_ptr(), s);
  }
  return result(status, y, codes, z, rstd);
  END_HANDLE_TH_ERRORS
}

// (function, x, w_gate, w_up, eps) -> (h, s, u, codes, z, rstd)
PyObject* norm_linear_swiglu_fwd(PyObject*, PyObject* const* a, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  at::Tensor x, wg, wu;
  int64_t m;
  c10::SmallVector<int64_t, 6> shape;
  if (n != 5 || !PyFloat_CheckExact(a[4]) || !plain(a[1], x) || !plain(a[2], wg) || !plain(a[3], wu) ||
      !layer(x, wg, m, shape) || !same(wu, wg) || wu.sizes() != wg.sizes())
    Py_RETURN_NONE;
  void* st;
  if (!stream_of(x, st)) return nullptr;
  at::Tensor h, s, u, codes, z, rstd;
  const auto f = address<int (*)(int, int64_t, int64_t, int64_t, float, const void*, const void*, const void*, void*,
                                 void*, void*, void*, void*, void*, void*, void*)>(a[0]);
  int status;
  {
    NoGil released;
    h = at::empty(shape, x.options());
    s = at::empty(shape, x.options());
    u = at::empty(shape, x.options());
    z = at::empty(x.sizes(), x.options());
    rstd = at::empty({m}, x.options().dtype(at::kFloat));
    codes = words(code_words(m * wg.size(0)), x);
    status = f(kBf16, m, wg.size(0), wg.size(1), float(PyFloat_AS_DOUBLE(a[4])), x.data_ptr(), wg.data_ptr(),
               wu.data_ptr(), h.data_ptr(), s.data_ptr(), u.data_ptr(), codes.data_ptr(), nullptr, z.data_ptr(),
               rstd.data_ptr(), st);
  }
  return result(status, h, s, u, codes, z, rstd);
  END_HANDLE_TH_ERRORS
}

// (torch's raw-stream accessor)
PyObject* bind(PyObject*, PyObject* accessor) {
  Py_INCREF(accessor);
  Py_XSETREF(g_raw_stream, accessor);
  Py_RETURN_NONE;
}

#define LMBP_FAST(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {LMBP_FAST(act_fwd), LMBP_FAST(act_bwd), LMBP_FAST(glu_fwd), LMBP_FAST(glu_bwd),
                          LMBP_FAST(norm_fwd), LMBP_FAST(norm_bwd), LMBP_FAST(linear_act_fwd),
                          LMBP_FAST(linear_swiglu_fwd), LMBP_FAST(norm_linear_act_fwd),
                          LMBP_FAST(norm_linear_swiglu_fwd), {"bind", bind, METH_O, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall() { return PyModule_Create(&kModule); }
