// The calls of one operation that a Python program makes once per layer, marshalled natively: argument checks, descriptor, output
// and workspace tensors, the call of the C ABI.  At small batches such a call is a few microseconds of GPU time, and what it
// costs in the interpreter (a tensor allocation 1.3 us, an address with its checks 0.3, a converted argument 0.1, five to fifteen
// of each) is longer: a float bottleneck block at batch 2, 21 calls, forward, backward and LARS, took 250 us for 188 us of GPU
// time with the same steps in Python, and takes 218 with them here.
// Signatures and defaults are those of the functions of the same names in binding.py, which are the callers.  Errors are raised as
// there (AssertionError, TypeError, ValueError, Rn50Error), and torch's own as torch raises them from Python (an allocation that
// does not fit: torch.OutOfMemoryError), without a C++ backtrace in the text.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <exception>
#include <string>
#include <vector>

#include <ATen/ATen.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../../include/rn50_hip.h"

namespace {

PyObject *g_error = nullptr, *g_stream = nullptr, *g_device = nullptr;  // Rn50Error; torch's current stream of a device and current device

struct PyError {  // (a Python exception is set)
};

// The call itself, without the interpreter's lock (a launch may have to wait for room in its queue).
template <typename F>
void call(F f) {
  PyThreadState* state = PyEval_SaveThread();
  const int rc = f();
  PyEval_RestoreThread(state);
  if (rc == 0) return;
  PyObject* e = PyObject_CallFunction(g_error, "is", rc, rn50_last_error());
  if (e) {
    PyErr_SetObject(g_error, e);
    Py_DECREF(e);
  }
  throw PyError();
}
[[noreturn]] void raise(PyObject* type, const char* text) {
  PyErr_SetString(type, text);
  throw PyError();
}

const at::Tensor* tensor(PyObject* o) {  // null: None
  if (o == Py_None) return nullptr;
  if (!THPVariable_Check(o)) raise(PyExc_TypeError, "expected a tensor");
  return &THPVariable_Unpack(o);
}
const at::Tensor& required(PyObject* o) {
  const at::Tensor* t = tensor(o);
  if (!t) raise(PyExc_TypeError, "expected a tensor");
  return *t;
}
template <typename T = void>
T* addr(const at::Tensor* t) {
  if (!t) return nullptr;
  if (!t->is_cuda() || !t->is_contiguous()) raise(PyExc_AssertionError, "device, contiguous tensors only");
  return static_cast<T*>(t->data_ptr());
}
template <typename T = void>
T* addr(const at::Tensor& t) { return addr<T>(&t); }

int dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::kFloat) return RN50_F32;
  if (t.scalar_type() == at::kBFloat16) return RN50_BF16;
  raise(PyExc_TypeError, (std::string("unsupported dtype ") + c10::toString(t.scalar_type())).c_str());
}
int to_int(PyObject* o) {
  const long v = PyLong_AsLong(o);
  if (v == -1 && PyErr_Occurred()) throw PyError();
  return static_cast<int>(v);
}
double to_double(PyObject* o) {
  const double v = PyFloat_AsDouble(o);
  if (v == -1.0 && PyErr_Occurred()) throw PyError();
  return v;
}
struct Shape4 {
  int64_t d[4];
};
Shape4 shape4(const at::Tensor& t) {
  if (t.dim() != 4) raise(PyExc_ValueError, "a tensor of four dimensions is expected");
  return {{t.size(0), t.size(1), t.size(2), t.size(3)}};
}
Shape4 shape4(PyObject* shape) {  // (any iterable of four numbers)
  Shape4 s;
  PyObject* seq = PySequence_Fast(shape, "a shape of four dimensions is expected");  // (a tuple or list is taken as it is)
  if (!seq) throw PyError();
  const Py_ssize_t n = PySequence_Fast_GET_SIZE(seq);
  for (Py_ssize_t i = 0; i < 4 && n == 4 && !PyErr_Occurred(); ++i) s.d[i] = PyLong_AsLongLong(PySequence_Fast_GET_ITEM(seq, i));
  Py_DECREF(seq);
  if (PyErr_Occurred()) throw PyError();
  if (n != 4) raise(PyExc_ValueError, "a shape of four dimensions is expected");
  return s;
}
rn50_conv_desc conv_desc(const Shape4& x, const Shape4& w, PyObject* stride, PyObject* pad, int dtype) {
  if (x.d[3] != w.d[3]) raise(PyExc_AssertionError, "channels of the input and of the weights");
  auto i = [](int64_t v) { return static_cast<int>(v); };
  return rn50_conv_desc{i(x.d[0]), i(x.d[1]), i(x.d[2]), i(x.d[3]), i(w.d[0]), i(w.d[1]), i(w.d[2]), to_int(stride), to_int(pad), dtype};
}
at::Tensor empty(at::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
  return at::empty(size, at::TensorOptions().dtype(type).device(like.device()));
}
// A workspace of at least `need` bytes; none is made where none is needed.
struct Workspace {
  at::Tensor made;
  void* p = nullptr;
  size_t bytes = 0;
  Workspace(PyObject* given, size_t need, const at::Tensor& like) {
    const at::Tensor* t = tensor(given);
    if (!t && need) {
      made = empty({static_cast<int64_t>(need)}, at::kByte, like);
      t = &made;
    }
    p = addr(t);
    bytes = t ? static_cast<size_t>(t->numel()) : 0;
  }
};
// The tensor that is given, or a new one.
at::Tensor output(PyObject* given, at::IntArrayRef size, at::ScalarType type, const at::Tensor& like) {
  const at::Tensor* t = tensor(given);
  return t ? *t : empty(size, type, like);
}
PyObject* wrap(const at::Tensor& t) { return THPVariable_Wrap(t); }

template <typename F>
PyObject* guarded(Py_ssize_t n, Py_ssize_t want, F f) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "%zd arguments expected, got %zd", want, n);
    return nullptr;
  }
  try {
    return f();
  } catch (const PyError&) {
    return nullptr;
  } catch (const std::exception&) {
    torch::translate_exception_to_python(std::current_exception());
    return nullptr;
  }
}
void* current_stream() {  // (asked for after the arguments were checked: without a GPU it raises)
  PyObject* dev = PyObject_CallNoArgs(g_device);
  if (!dev) throw PyError();
  PyObject* num = PyObject_CallOneArg(g_stream, dev);
  Py_DECREF(dev);
  if (!num) throw PyError();
  void* s = PyLong_AsVoidPtr(num);
  Py_DECREF(num);
  if (!s && PyErr_Occurred()) throw PyError();
  return s;
}

// conv_fwd(x, w, stride, pad, y, workspace)
PyObject* conv_fwd_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 6, [&]() -> PyObject* {
    const at::Tensor &x = required(a[0]), &w = required(a[1]);
    const rn50_conv_desc d = conv_desc(shape4(x), shape4(w), a[2], a[3], dtype_of(x));
    if (d.stride == 0) raise(PyExc_ZeroDivisionError, "stride");
    auto extent = [&](int64_t span) { return (span >= 0 ? span / d.stride : -1 - (-1 - span) / d.stride) + 1; };
    const at::Tensor y = output(a[4], {d.N, extent(d.H + 2 * d.pad - d.R), extent(d.W + 2 * d.pad - d.S), d.Cout}, x.scalar_type(), x);
    const Workspace ws(a[5], a[5] == Py_None ? conv_fwd_workspace_bytes(&d) : 0, x);
    void* const p[] = {addr(x), addr(w), addr(y), current_stream()};
    call([&] { return conv_fwd(&d, p[0], p[1], p[2], ws.p, ws.bytes, p[3]); });
    return wrap(y);
  });
}
// conv_dgrad(dy, w, x_shape, stride, pad, dx, workspace)
PyObject* conv_dgrad_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const at::Tensor &dy = required(a[0]), &w = required(a[1]);
    const Shape4 xs = shape4(a[2]);
    const rn50_conv_desc d = conv_desc(xs, shape4(w), a[3], a[4], dtype_of(dy));
    const at::Tensor dx = output(a[5], {xs.d, 4}, dy.scalar_type(), dy);
    const Workspace ws(a[6], a[6] == Py_None ? conv_dgrad_workspace_bytes(&d) : 0, dy);
    void* const p[] = {addr(dy), addr(w), addr(dx), current_stream()};
    call([&] { return conv_dgrad(&d, p[0], p[1], p[2], ws.p, ws.bytes, p[3]); });
    return wrap(dx);
  });
}
// conv_wgrad(x, dy, w_shape, stride, pad, dw, workspace)
PyObject* conv_wgrad_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 7, [&]() -> PyObject* {
    const at::Tensor &x = required(a[0]), &dy = required(a[1]);
    const Shape4 ws_ = shape4(a[2]);
    const rn50_conv_desc d = conv_desc(shape4(x), ws_, a[3], a[4], dtype_of(x));
    const at::Tensor dw = output(a[5], {ws_.d, 4}, at::kFloat, x);
    const Workspace ws(a[6], a[6] == Py_None ? conv_wgrad_workspace_bytes(&d) : 0, x);
    void* const p[] = {addr(x), addr(dy), addr(dw), current_stream()};
    call([&] { return conv_wgrad(&d, p[0], p[1], static_cast<float*>(p[2]), ws.p, ws.bytes, p[3]); });
    return wrap(dw);
  });
}
rn50_bn_desc bn_desc(const at::Tensor& x, PyObject* eps, PyObject* mode) {
  const int64_t C = x.size(-1);
  if (x.dim() != 4 && C == 0) raise(PyExc_ZeroDivisionError, "channels");
  rn50_bn_desc d{1, 1, static_cast<int>(C ? x.numel() / C : 0), static_cast<int>(C), static_cast<float>(to_double(eps)), dtype_of(x), to_int(mode)};
  if (x.dim() == 4) {
    d.N = static_cast<int>(x.size(0)); d.H = static_cast<int>(x.size(1)); d.W = static_cast<int>(x.size(2));
  }
  return d;
}
// bn_relu_fwd(x, gamma, beta, residual, eps, mode, running_mean, running_var, momentum, workspace, relu_mask)
PyObject* bn_relu_fwd_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 11, [&]() -> PyObject* {
    const at::Tensor& x = required(a[0]);
    const rn50_bn_desc d = bn_desc(x, a[4], a[5]);
    const at::Tensor y = at::empty_like(x), mean = empty({d.C}, at::kFloat, x), rstd = empty({d.C}, at::kFloat, x);
    const Workspace ws(a[9], a[9] == Py_None ? bn_relu_fwd_workspace_bytes(&d) : 0, x);
    const float momentum = static_cast<float>(to_double(a[8]));
    float* const f[] = {addr<float>(tensor(a[1])), addr<float>(tensor(a[2])), addr<float>(mean), addr<float>(rstd),
                        addr<float>(tensor(a[6])), addr<float>(tensor(a[7]))};
    uint8_t* const mask = addr<uint8_t>(tensor(a[10]));
    void* const p[] = {addr(x), addr(tensor(a[3])), addr(y), current_stream()};
    call([&] { return bn_relu_fwd(&d, p[0], f[0], f[1], p[1], p[2], mask, f[2], f[3], f[4], f[5], momentum, ws.p, ws.bytes, p[3]); });
    return Py_BuildValue("NNN", wrap(y), wrap(mean), wrap(rstd));
  });
}
// bn_relu_bwd(dz, x, z, gamma, mean, rstd, mode, beta, dz2, eps, workspace, relu_mask)
PyObject* bn_relu_bwd_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 12, [&]() -> PyObject* {
    const at::Tensor& x = required(a[1]);
    const rn50_bn_desc d = bn_desc(x, a[9], a[6]);
    const at::Tensor dx = at::empty_like(x);
    at::Tensor dres;
    if (d.mode == 2) dres = at::empty_like(x);
    const at::Tensor dgamma = empty({d.C}, at::kFloat, x), dbeta = empty({d.C}, at::kFloat, x);
    const Workspace ws(a[10], a[10] == Py_None ? bn_relu_bwd_workspace_bytes(&d) : 0, x);
    float* const f[] = {addr<float>(tensor(a[3])), addr<float>(tensor(a[7])), addr<float>(tensor(a[4])), addr<float>(tensor(a[5])),
                        addr<float>(dgamma), addr<float>(dbeta)};
    uint8_t* const mask = addr<uint8_t>(tensor(a[11]));
    void* const p[] = {addr(tensor(a[0])), addr(tensor(a[8])), addr(x), addr(tensor(a[2])), addr(dx),
                       dres.defined() ? addr(dres) : nullptr, current_stream()};
    call([&] {
      return bn_relu_bwd(&d, p[0], p[1], p[2], p[3], mask, f[0], f[1], f[2], f[3], p[4], p[5], f[4], f[5], ws.p, ws.bytes, p[6]);
    });
    PyObject* res = Py_None;
    if (d.mode == 2) res = wrap(dres); else Py_INCREF(Py_None);
    return Py_BuildValue("NNNN", wrap(dx), res, wrap(dgamma), wrap(dbeta));
  });
}
// setup(Rn50Error, current raw stream of a device, current device)
PyObject* setup_py(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return guarded(n, 3, [&]() -> PyObject* {
    PyObject** const kept[] = {&g_error, &g_stream, &g_device};
    for (int i = 0; i < 3; ++i) {
      Py_INCREF(a[i]);
      Py_XSETREF(*kept[i], a[i]);
    }
    Py_RETURN_NONE;
  });
}

#define FAST(name, f) {name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {FAST("conv_fwd", conv_fwd_py), FAST("conv_dgrad", conv_dgrad_py), FAST("conv_wgrad", conv_wgrad_py),
                          FAST("bn_relu_fwd", bn_relu_fwd_py), FAST("bn_relu_bwd", bn_relu_bwd_py),
                          FAST("setup", setup_py), {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_ops", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__ops() { return PyModule_Create(&kModule); }
