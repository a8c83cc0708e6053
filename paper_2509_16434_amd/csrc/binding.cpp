// The calls a training program makes once per environment step (buffer_write, act, buffer_write_outcome, gae), bound
// natively: argument checks and the call into libppo_learner.so in 0.4 us, where checking seven tensors through
// Python attributes and calling through ctypes cost 3.4 us beside the kernel launch behind it, which set the pace of
// small tasks (64 environments: 16 writes, 145 .. 161 -> 110 .. 114 us).  Marshalling only: the library's functions are
// handed in as addresses by learner.py, which loads the library and binds everything else.
#include <torch/csrc/autograd/python_variable.h>
#include <ATen/ATen.h>

#include "../../include/ppo_learner.h"

namespace {

decltype(&ppo_buffer_write) f_write = nullptr;
decltype(&ppo_buffer_write_range) f_write_range = nullptr;
decltype(&ppo_act) f_act = nullptr;
decltype(&ppo_buffer_write_outcome) f_outcome = nullptr;
decltype(&ppo_gae) f_gae = nullptr;

const char* dtype_name(at::ScalarType t) {
  return t == at::kFloat ? "torch.float32" : t == at::kBFloat16 ? "torch.bfloat16" : t == at::kByte ? "torch.uint8" : at::toString(t);
}

// Device pointer of a contiguous CUDA tensor of `numel` elements of type `dt`; None gives NULL.  False: error set.
bool device_ptr(PyObject* o, at::ScalarType dt, int64_t numel, void** out) {
  *out = nullptr;
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) { PyErr_Format(PyExc_TypeError, "expected a torch.Tensor or None, got %s", Py_TYPE(o)->tp_name); return false; }
  try {  // a tensor without storage of its own (a tracer's stand-in) throws when asked for its address
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda() || !t.is_contiguous()) { PyErr_SetString(PyExc_ValueError, "expected a contiguous CUDA tensor"); return false; }
    if (t.scalar_type() != dt) { PyErr_Format(PyExc_ValueError, "expected dtype %s, got %s", dtype_name(dt), dtype_name(t.scalar_type())); return false; }
    if (t.numel() != numel) { PyErr_Format(PyExc_ValueError, "expected %lld elements, got %lld", (long long)numel, (long long)t.numel()); return false; }
    *out = t.data_ptr();
    return true;
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return false;
  }
}

bool integers(PyObject* const* args, int n, long long* out) {
  for (int i = 0; i < n; ++i) {
    PyObject* x = PyNumber_Index(args[i]);  // any integer type; a float is a TypeError, as it is through ctypes
    if (!x) return false;
    out[i] = PyLong_AsLongLong(x);
    Py_DECREF(x);
    if (out[i] == -1 && PyErr_Occurred()) return false;
  }
  return true;
}

bool arity(Py_ssize_t got, Py_ssize_t want, const char* name) {
  if (got == want) return true;
  PyErr_Format(PyExc_TypeError, "%s takes %zd arguments, got %zd", name, want, got);
  return false;
}

// setup(addresses of ppo_buffer_write, ppo_buffer_write_range, ppo_act, ppo_buffer_write_outcome, ppo_gae)
PyObject* py_setup(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long long v[5];
  if (!arity(n, 5, "setup") || !integers(a, 5, v)) return nullptr;
  f_write = reinterpret_cast<decltype(f_write)>(v[0]); f_write_range = reinterpret_cast<decltype(f_write_range)>(v[1]);
  f_act = reinterpret_cast<decltype(f_act)>(v[2]); f_outcome = reinterpret_cast<decltype(f_outcome)>(v[3]); f_gae = reinterpret_cast<decltype(f_gae)>(v[4]);
  Py_RETURN_NONE;
}

// write(handle, fp32 images, elements per observation, P, A, t, env_offset or -1, count, obs, proprio, action, logp, value, reward, done) -> code
PyObject* py_write(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long long v[8];
  if (!arity(n, 15, "write") || !integers(a, 8, v)) return nullptr;
  const long long cnt = v[7];
  void* p[7];
  if (!device_ptr(a[8], v[1] ? at::kFloat : at::kBFloat16, cnt * v[2], &p[0]) || !device_ptr(a[9], at::kFloat, cnt * v[3], &p[1]) ||
      !device_ptr(a[10], at::kFloat, cnt * v[4], &p[2]) || !device_ptr(a[11], at::kFloat, cnt, &p[3]) || !device_ptr(a[12], at::kFloat, cnt, &p[4]) ||
      !device_ptr(a[13], at::kFloat, cnt, &p[5]) || !device_ptr(a[14], at::kByte, cnt, &p[6]))
    return nullptr;
  ppo_ctx* c = reinterpret_cast<ppo_ctx*>(v[0]);
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  if (v[6] < 0)
    rc = f_write(c, (int32_t)v[5], p[0], (const float*)p[1], (const float*)p[2], (const float*)p[3], (const float*)p[4], (const float*)p[5], (const uint8_t*)p[6]);
  else
    rc = f_write_range(c, (int32_t)v[5], (int32_t)v[6], (int32_t)cnt, p[0], (const float*)p[1], (const float*)p[2], (const float*)p[3], (const float*)p[4],
                       (const float*)p[5], (const uint8_t*)p[6]);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

// act(handle, fp32 images, elements per observation, P, A, t, N, obs, proprio, noise) -> (code, action [N][A], logp [N], value [N])
PyObject* py_act(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long long v[7];
  if (!arity(n, 10, "act") || !integers(a, 7, v)) return nullptr;
  const long long N = v[6];
  void* p[3];
  if (!device_ptr(a[7], v[1] ? at::kFloat : at::kBFloat16, N * v[2], &p[0]) || !device_ptr(a[8], at::kFloat, N * v[3], &p[1]) ||
      !device_ptr(a[9], at::kFloat, N * v[4], &p[2]))
    return nullptr;
  try {
    const auto opt = at::TensorOptions().dtype(at::kFloat).device(at::kCUDA);
    at::Tensor action = at::empty({N, v[4]}, opt), logp = at::empty({N}, opt), value = at::empty({N}, opt);
    int rc;
    Py_BEGIN_ALLOW_THREADS;
    rc = f_act(reinterpret_cast<ppo_ctx*>(v[0]), (int32_t)v[5], p[0], (const float*)p[1], (const float*)p[2], (float*)action.data_ptr(), (float*)logp.data_ptr(),
               (float*)value.data_ptr());
    Py_END_ALLOW_THREADS;
    return Py_BuildValue("iNNN", rc, THPVariable_Wrap(std::move(action)), THPVariable_Wrap(std::move(logp)), THPVariable_Wrap(std::move(value)));
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// outcome(handle, t, N, reward, done) -> code
PyObject* py_outcome(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long long v[3];
  void* p[2];
  if (!arity(n, 5, "outcome") || !integers(a, 3, v) || !device_ptr(a[3], at::kFloat, v[2], &p[0]) || !device_ptr(a[4], at::kByte, v[2], &p[1])) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = f_outcome(reinterpret_cast<ppo_ctx*>(v[0]), (int32_t)v[1], (const float*)p[0], (const uint8_t*)p[1]);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

// gae(handle, N, last_value, gamma, lambda) -> code
PyObject* py_gae(PyObject*, PyObject* const* a, Py_ssize_t n) {
  long long v[2];
  void* p;
  if (!arity(n, 5, "gae") || !integers(a, 2, v) || !device_ptr(a[2], at::kFloat, v[1], &p)) return nullptr;
  const double gamma = PyFloat_AsDouble(a[3]), lam = PyFloat_AsDouble(a[4]);
  if (PyErr_Occurred()) return nullptr;
  int rc;
  Py_BEGIN_ALLOW_THREADS;
  rc = f_gae(reinterpret_cast<ppo_ctx*>(v[0]), (const float*)p, (float)gamma, (float)lam);
  Py_END_ALLOW_THREADS;
  return PyLong_FromLong(rc);
}

PyMethodDef methods[] = {{"setup", (PyCFunction)(void*)py_setup, METH_FASTCALL, nullptr}, {"write", (PyCFunction)(void*)py_write, METH_FASTCALL, nullptr},
                         {"act", (PyCFunction)(void*)py_act, METH_FASTCALL, nullptr}, {"outcome", (PyCFunction)(void*)py_outcome, METH_FASTCALL, nullptr},
                         {"gae", (PyCFunction)(void*)py_gae, METH_FASTCALL, nullptr}, {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding() { return PyModule_Create(&module); }
