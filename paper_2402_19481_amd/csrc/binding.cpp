// The operations of __init__.py that a caller issues one by one, bound natively: a few kernels of some microseconds each are waited for
// less than they take to issue.  Marshalling only: checks that a tensor is one the library can take, allocates the result with torch,
// and calls the C entry point on the current stream, with the interpreter released.  Per call ctypes and Python took 7 - 8 us of the host
// beside the launch, this 2; three calls of a small float32 block 30 -> 20 us.  The entry points are addresses that __init__.py hands over
// (of the library that it has loaded).
#include <Python.h>

#include <ATen/ops/empty.h>
#include <ATen/ops/empty_like.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

namespace {

enum { kF32 = 0, kBF16 = 1 };
PyObject *g_error = nullptr, *g_torch_memory = nullptr, *g_torch_device = nullptr;   // DfError, torch.OutOfMemoryError, torch.AcceleratorError
const char* (*g_strerror)(int) = nullptr;

struct Failed {};                                      // a Python exception is set

[[noreturn]] void fail(PyObject* kind, const char* text) {
  PyErr_SetString(kind, text);
  throw Failed{};
}
const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_Check(o)) fail(PyExc_TypeError, "expected a tensor");
  return THPVariable_Unpack(o);
}
// Device pointer of a tensor, nullptr for None
void* ptr(PyObject* o) {
  if (o == Py_None) return nullptr;
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || !t.is_contiguous()) fail(g_error, "tensors must be contiguous and on the GPU");
  return t.data_ptr();
}
int dtype(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return kF32;
  if (t.scalar_type() == at::kBFloat16) return kBF16;
  PyErr_Format(g_error, "unsupported dtype torch.%s", t.scalar_type() == at::kHalf ? "float16" : c10::toString(t.scalar_type()));
  throw Failed{};
}
long long integer(PyObject* o) {
  const long long v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw Failed{};
  return v;
}
int int32(PyObject* o) {
  const long long v = integer(o);
  if (v != (int)v) fail(PyExc_OverflowError, "integer out of range");
  return (int)v;
}
float real(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw Failed{};
  return (float)v;
}
void dims(const at::Tensor& t, int64_t n, const char* text) {
  if (t.dim() != n) fail(PyExc_ValueError, text);
}
// `what` divided by a caller's number, as Python's // and with its exception
long long over(long long what, long long by) {
  if (by == 0) fail(PyExc_ZeroDivisionError, "integer division or modulo by zero");
  const long long q = what / by;
  return q * by != what && (what < 0) != (by < 0) ? q - 1 : q;
}
int small(long long v) {                               // (the C entry points refuse what is not positive)
  return v > 0x7fffffffLL ? fail(PyExc_OverflowError, "size out of range"), 0 : (int)v;
}
void* stream() { return (void*)c10::hip::getCurrentHIPStream().stream(); }
void check(int rc) {
  if (rc == 0) return;
  PyErr_Format(g_error, "libdistrifusion: %s (%d)", g_strerror(rc), rc);
  throw Failed{};
}
template <typename F>
PyObject* guarded(F f) {
  try {
    return f();
  } catch (const Failed&) {
    return nullptr;
  } catch (python_error& e) {
    e.restore();
  } catch (const c10::OutOfMemoryError& e) {           // (as torch raises them: its own translation is not exported)
    PyErr_SetString(g_torch_memory, e.what_without_backtrace());
  } catch (const c10::AcceleratorError& e) {
    PyErr_SetString(g_torch_device, e.what_without_backtrace());
  } catch (const c10::Error& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what_without_backtrace());
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}
#define DF_ARGS(n) \
  if (na != (n)) { PyErr_SetString(PyExc_TypeError, "wrong number of arguments"); return nullptr; }
// The interpreter is released while torch allocates (its allocator may have to wait for others) and the library launches
struct Released {
  PyThreadState* state = PyEval_SaveThread();
  ~Released() { PyEval_RestoreThread(state); }
};

using GnFn = int (*)(const void*, void*, const float*, float*, const float*, const float*, int, int, int, int, int, int, int, float, int, int,
                     int, void*);
using ConvFn = int (*)(const void*, const void*, const void*, const float*, void*, int, int, int, int, int, int, int, int, int, int, int, void*);
using AttnFn = int (*)(const void*, const void*, const void*, const void*, const void*, void*, int, int, int, int, int, int, float, int, void*);
using AttnAxisFn = int (*)(const void*, const void*, const void*, const void*, const void*, void*, int, int, int, int, int, int, int, float, int,
                           int, void*);
using LinearFn = int (*)(const void*, const void*, const float*, const float*, void*, int, int, int, int, void*);
using RefreshFn = int (*)(void*, const void*, int, long long, int, int, int, void*);
GnFn g_gn;
ConvFn g_conv;
AttnFn g_attn;
AttnAxisFn g_attn_axis;
LinearFn g_linear;
RefreshFn g_refresh;

// setup(DfError, torch.OutOfMemoryError, torch.AcceleratorError, addresses of df_strerror, df_groupnorm_stale, df_conv3x3_halo_axis,
// df_attn_displaced, df_attn_displaced_axis, df_linear, df_buffer_refresh)
PyObject* setup(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(10)
  return guarded([&]() -> PyObject* {
    void* f[7];
    for (int i = 0; i < 7; ++i) f[i] = (void*)integer(a[i + 3]);
    PyObject** const kinds[] = {&g_error, &g_torch_memory, &g_torch_device};
    for (int i = 0; i < 3; ++i) {
      Py_INCREF(a[i]);
      Py_XDECREF(*kinds[i]);
      *kinds[i] = a[i];
    }
    g_strerror = (const char* (*)(int))f[0];
    g_gn = (GnFn)f[1]; g_conv = (ConvFn)f[2]; g_attn = (AttnFn)f[3]; g_attn_axis = (AttnAxisFn)f[4]; g_linear = (LinearFn)f[5];
    g_refresh = (RefreshFn)f[6];
    Py_RETURN_NONE;
  });
}

// x_fresh, stale_stats, gamma, beta, G, patch_idx, N, eps, stat_mode, fuse_silu, fresh_stats_out or None -> (y, fresh_stats)
PyObject* groupnorm_stale(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(11)
  return guarded([&] {
    const at::Tensor& x = tensor(a[0]);
    dims(x, 4, "x_fresh: expected [B, R, W, C]");
    const int G = int32(a[4]), patch = int32(a[5]), N = int32(a[6]), mode = int32(a[8]), silu = int32(a[9]);
    const float eps = real(a[7]);
    const void *xp = ptr(a[0]), *st = ptr(a[1]), *gm = ptr(a[2]), *bt = ptr(a[3]);
    void* fp = ptr(a[10]);
    const int dt = dtype(x), B = small(x.size(0)), R = small(x.size(1)), W = small(x.size(2)), C = small(x.size(3));
    at::Tensor y, fs;
    int rc;
    {
      Released r;
      y = at::empty_like(x);
      if (a[10] == Py_None) {
        fs = at::empty({B, G, 2}, x.options().dtype(at::kFloat));
        fp = fs.data_ptr();
      }
      rc = g_gn(xp, y.data_ptr(), (const float*)st, (float*)fp, (const float*)gm, (const float*)bt, B, R, W, C, G, patch, N, eps, mode, silu, dt,
                stream());
    }
    check(rc);
    PyObject* fo = a[10] == Py_None ? THPVariable_Wrap(std::move(fs)) : Py_NewRef(a[10]);
    PyObject* yo = THPVariable_Wrap(std::move(y));
    PyObject* t = PyTuple_Pack(2, yo, fo);
    Py_XDECREF(yo);
    Py_XDECREF(fo);
    return t;
  });
}

// x_fresh, stale_full, w, bias, patch_idx, N, stride, act, axis -> y
PyObject* conv3x3_halo(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(9)
  return guarded([&] {
    const at::Tensor &x = tensor(a[0]), &w = tensor(a[2]);
    dims(x, 4, "x_fresh: expected [B, R, W, Cin]");
    if (w.dim() < 1) fail(PyExc_ValueError, "w: expected [Cout, 3, 3, Cin]");
    const int patch = int32(a[4]), N = int32(a[5]), stride = int32(a[6]), act = int32(a[7]), axis = int32(a[8]);
    const long long Ro = over(x.size(1), stride), Wo = over(x.size(2), stride);
    const void *xp = ptr(a[0]), *sp = ptr(a[1]), *wp = ptr(a[2]), *bp = ptr(a[3]);
    const int dt = dtype(x), B = small(x.size(0)), Cin = small(x.size(3)), Cout = small(w.size(0));
    const int H = small(x.size(1) * (axis == 0 ? N : 1)), W = small(x.size(2) * (axis == 0 ? 1 : N));
    at::Tensor y;
    int rc;
    {
      Released r;
      y = at::empty({B, Ro, Wo, Cout}, x.options());
      rc = g_conv(xp, sp, wp, (const float*)bp, y.data_ptr(), B, H, W, Cin, Cout, patch, N, stride, act, dt, axis, stream());
    }
    check(rc);
    return THPVariable_Wrap(std::move(y));
  });
}

// q, k_fresh, v_fresh, k_stale, v_stale, heads, patch_idx, N, scale or None, out or None -> out
PyObject* attn_displaced(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(10)
  return guarded([&] {
    const at::Tensor& q = tensor(a[0]);
    dims(q, 3, "q: expected [B, Lq, C]");
    const int heads = int32(a[5]), patch = int32(a[6]), N = int32(a[7]);
    const long long d = over(q.size(2), heads);
    const float scale = a[8] == Py_None ? (float)std::pow((double)d, -0.5) : real(a[8]);
    const void *qp = ptr(a[0]), *kf = ptr(a[1]), *vf = ptr(a[2]), *ks = ptr(a[3]), *vs = ptr(a[4]);
    void* op = ptr(a[9]);
    const int dt = dtype(q), B = small(q.size(0)), L = small(q.size(1) * N), hd = small(d);
    at::Tensor out;
    int rc;
    {
      Released r;
      if (a[9] == Py_None) {
        out = at::empty_like(q);
        op = out.data_ptr();
      }
      rc = g_attn(qp, kf, vf, ks, vs, op, B, L, heads, hd, patch, N, scale, dt, stream());
    }
    check(rc);
    return a[9] == Py_None ? THPVariable_Wrap(std::move(out)) : Py_NewRef(a[9]);
  });
}

// q, k_fresh, v_fresh, k_stale, v_stale, heads, H, W, patch_idx, N, scale or None, axis -> out
PyObject* attn_displaced_axis(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(12)
  return guarded([&] {
    const at::Tensor& q = tensor(a[0]);
    dims(q, 3, "q: expected [B, Lq, C]");
    const int heads = int32(a[5]), H = int32(a[6]), W = int32(a[7]), patch = int32(a[8]), N = int32(a[9]), axis = int32(a[11]);
    const long long d = over(q.size(2), heads);
    const float scale = a[10] == Py_None ? (float)std::pow((double)d, -0.5) : real(a[10]);
    const void *qp = ptr(a[0]), *kf = ptr(a[1]), *vf = ptr(a[2]), *ks = ptr(a[3]), *vs = ptr(a[4]);
    const int dt = dtype(q), B = small(q.size(0)), hd = small(d);
    at::Tensor out;
    int rc;
    {
      Released r;
      out = at::empty_like(q);
      rc = g_attn_axis(qp, kf, vf, ks, vs, out.data_ptr(), B, H, W, heads, hd, patch, N, scale, dt, axis, stream());
    }
    check(rc);
    return THPVariable_Wrap(std::move(out));
  });
}

// x, w, bias, residual, out or None, dtype of a new out (0 float32, 1 bf16) -> out
PyObject* linear(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(6)
  return guarded([&] {
    const at::Tensor &x = tensor(a[0]), &w = tensor(a[1]);
    dims(x, 2, "x: expected [M, K]");
    if (w.dim() < 1) fail(PyExc_ValueError, "w: expected [N, K]");
    const void *xp = ptr(a[0]), *wp = ptr(a[1]), *bp = ptr(a[2]), *rp = ptr(a[3]);
    void* op = ptr(a[4]);
    const int dt = a[4] != Py_None ? dtype(tensor(a[4])) : int32(a[5]), M = small(x.size(0)), Nn = small(w.size(0)), K = small(x.size(1));
    at::Tensor out;
    int rc;
    {
      Released r;
      if (a[4] == Py_None) {
        out = at::empty({M, Nn}, x.options().dtype(dt == kF32 ? at::kFloat : at::kBFloat16));
        op = out.data_ptr();
      }
      rc = g_linear(xp, wp, (const float*)bp, (const float*)rp, op, M, Nn, K, dt, stream());
    }
    check(rc);
    return a[4] == Py_None ? THPVariable_Wrap(std::move(out)) : Py_NewRef(a[4]);
  });
}

// dst_full, src_patch, patch_idx, N -> dst_full
PyObject* buffer_refresh(PyObject*, PyObject* const* a, Py_ssize_t na) {
  DF_ARGS(4)
  return guarded([&] {
    const at::Tensor& t = tensor(a[0]);
    if (t.dim() < 1) fail(PyExc_ValueError, "dst_full: expected [B, ...]");
    const int patch = int32(a[2]), N = int32(a[3]), B = small(t.size(0));
    void *dp = ptr(a[0]), *sp = ptr(a[1]);
    const long long per = over(t.numel(), B);
    const int dt = dtype(t);
    int rc;
    {
      Released r;
      rc = g_refresh(dp, sp, B, per, patch, N, dt, stream());
    }
    check(rc);
    return Py_NewRef(a[0]);
  });
}

#define DF_METHOD(name) {#name, (PyCFunction)(void (*)(void))name, METH_FASTCALL, nullptr}
PyMethodDef methods[] = {DF_METHOD(setup),  DF_METHOD(groupnorm_stale), DF_METHOD(conv3x3_halo), DF_METHOD(attn_displaced), DF_METHOD(attn_displaced_axis),
                         DF_METHOD(linear), DF_METHOD(buffer_refresh), {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
