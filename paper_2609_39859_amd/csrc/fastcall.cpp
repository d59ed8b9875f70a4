// Python calls into libforkstep.so without the interpreter's share of the
// argument marshalling.
//
// A small step or training call takes a few microseconds on the GPU, and
// checking a dozen tensors attribute by attribute and filling a ctypes
// structure took longer than that (13.8 us per fork_grpo_objective, 13.5 us
// per fork_select, 18 us per small fork_step_ex).  Each function here makes
// the checks of _binding.py on the tensors themselves, fills the C structure
// and calls the library with the interpreter lock released.  It returns the
// library's return code, or None for any argument that is not of the plainest
// form or fails a check: _binding.py then goes through its own checks, which
// raise the error that describes it.
#include <Python.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "fork_step.h"

namespace {

int (*g_step_ex)(const fork_step_args*);
int (*g_step_noalloc)(const fork_step_args*);
int (*g_logprob)(const fork_logprob_args*);
int (*g_grpo)(const fork_grpo_args*);
int (*g_select)(const fork_select_args*);
int (*g_top)(const float*, int32_t, int32_t, int32_t, uint8_t*, void*);
PyObject* g_raw_stream;  // torch._C._cuda_getCurrentRawStream

// An argument that the plain path does not take.
struct Other {};

const at::Tensor& tensor(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw Other();
  return THPVariable_Unpack(o);
}

// Device pointer of a contiguous tensor of `n` elements on device `dev`.
void* ptr(PyObject* o, at::ScalarType type, int64_t n, int dev) {
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || t.get_device() != dev || t.scalar_type() != type || t.numel() != n ||
      !t.is_contiguous())
    throw Other();
  return t.data_ptr();
}

void* opt(PyObject* o, at::ScalarType type, int64_t n, int dev) {
  return o == Py_None ? nullptr : ptr(o, type, n, dev);
}

int32_t i32(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw Other();
  int overflow = 0;
  const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow || v < INT32_MIN || v > INT32_MAX) throw Other();
  return (int32_t)v;
}

int32_t size32(int64_t v) {
  if (v > INT32_MAX) throw Other();
  return (int32_t)v;
}

float f32(PyObject* o) {
  if (!PyFloat_CheckExact(o)) throw Other();
  return (float)PyFloat_AS_DOUBLE(o);
}

uint64_t bits(PyObject* o) {
  if (!PyLong_CheckExact(o)) throw Other();
  return PyLong_AsUnsignedLongLongMask(o);
}

// The given stream's handle, or the device's current stream's.
void* stream(PyObject* s, int dev) {
  PyObject* v;
  if (s == Py_None) {
    PyObject* d = PyLong_FromLong(dev);
    v = d ? PyObject_CallFunctionObjArgs(g_raw_stream, d, nullptr) : nullptr;
    Py_XDECREF(d);
  } else {
    v = PyObject_GetAttrString(s, "cuda_stream");
  }
  if (!v) {
    PyErr_Clear();
    throw Other();
  }
  void* p = PyLong_AsVoidPtr(v);
  Py_DECREF(v);
  if (PyErr_Occurred()) {
    PyErr_Clear();
    throw Other();
  }
  return p;
}

constexpr auto kF = at::ScalarType::Float;
constexpr auto kI = at::ScalarType::Int;
constexpr auto kB = at::ScalarType::Byte;

int32_t dtype_of(const at::Tensor& t) {
  if (t.scalar_type() == at::ScalarType::BFloat16) return FORK_BF16;
  if (t.scalar_type() == kF) return FORK_F32;
  throw Other();
}

// hidden [M, d] and W_head [V, d]
const at::Tensor& matrix(PyObject* o) {
  const at::Tensor& t = tensor(o);
  if (t.dim() != 2 || !t.is_cuda()) throw Other();
  return t;
}

void workspace(PyObject* o, int dev, void** p, size_t* n) {
  if (o == Py_None) return;
  const at::Tensor& t = tensor(o);
  if (!t.is_cuda() || t.get_device() != dev || !t.is_contiguous()) throw Other();
  *p = t.data_ptr();
  *n = (size_t)t.numel() * t.element_size();
}

template <class F, class A>
PyObject* call(F fn, const A& a) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(&a);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// Runs `f`; None for what the plain path does not take.
template <class F>
PyObject* plain(Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return nullptr;
  }
  try {
    return f();
  } catch (...) {
    // Other, or a tensor without storage of its own
  }
  Py_RETURN_NONE;
}

PyObject* step(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 27, [&] {
    fork_step_args a = {};
    const at::Tensor& h = matrix(v[1]);
    const at::Tensor& w = matrix(v[2]);
    const int dev = h.get_device();
    const int64_t d = h.size(1), V = w.size(0), M = h.size(0);
    a.block_len = i32(v[6]);
    a.B = i32(v[12]);
    a.L = i32(v[13]);
    if (M != (int64_t)a.B * a.L) throw Other();
    a.d = size32(d);
    a.V = size32(V);
    a.dtype = dtype_of(h);
    a.hidden = ptr(v[1], h.scalar_type(), M * d, dev);
    a.W_head = ptr(v[2], h.scalar_type(), V * d, dev);
    a.tokens = (int32_t*)ptr(v[3], kI, M, dev);
    a.mask = (uint8_t*)ptr(v[4], kB, M, dev);
    a.block_start = (int32_t*)ptr(v[5], kI, a.B, dev);
    a.tau = f32(v[7]);
    a.out_conf = (float*)ptr(v[8], kF, M, dev);
    a.out_entropy = (float*)ptr(v[9], kF, M, dev);
    a.out_logp = (float*)ptr(v[10], kF, M, dev);
    a.out_fallback = (int32_t*)ptr(v[11], kI, a.B, dev);
    a.out_lse = (float*)opt(v[14], kF, M, dev);
    a.out_argmax = (int32_t*)opt(v[15], kI, M, dev);
    a.out_ncommit = (int32_t*)opt(v[16], kI, a.B, dev);
    a.out_commit_pos = (int32_t*)opt(v[17], kI, (int64_t)a.B * a.block_len, dev);
    a.rule = i32(v[18]);
    workspace(v[19], dev, &a.workspace, &a.workspace_bytes);
    a.stream = stream(v[20], dev);
    if (v[21] != Py_None) throw Other();  // timing events
    a.fallback_uniform = (const float*)opt(v[22], kF, a.B, dev);
    a.rows_mode = i32(v[23]);
    a.sample_temperature = f32(v[24]);
    a.sample_seed = bits(v[25]);
    a.sample_counter = (uint32_t)bits(v[26]);
    return call(v[0] == Py_True ? g_step_noalloc : g_step_ex, a);
  });
}

PyObject* logprob(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 11, [&] {
    fork_logprob_args a = {};
    const at::Tensor& h = matrix(v[0]);
    const at::Tensor& w = matrix(v[1]);
    const int dev = h.get_device();
    const int64_t d = h.size(1), V = w.size(0), M = h.size(0), n = tensor(v[2]).numel();
    a.n = size32(n);
    a.M = size32(M);
    a.d = size32(d);
    a.V = size32(V);
    a.dtype = dtype_of(h);
    a.hidden = ptr(v[0], h.scalar_type(), M * d, dev);
    a.W_head = ptr(v[1], h.scalar_type(), V * d, dev);
    a.tokens = (const int32_t*)ptr(v[2], kI, n, dev);
    a.out_logp = (float*)ptr(v[3], kF, n, dev);
    a.rows = (const int32_t*)opt(v[4], kI, n, dev);
    a.out_q = (float*)opt(v[5], kF, n, dev);
    a.out_entropy = (float*)opt(v[6], kF, n, dev);
    a.out_lse = (float*)opt(v[7], kF, n, dev);
    if (v[8] != Py_None) throw Other();  // a caller workspace is not checked here
    a.stream = stream(v[9], dev);
    if (v[10] != Py_None) throw Other();  // timing events
    return call(g_logprob, a);
  });
}

PyObject* grpo(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 14, [&] {
    fork_grpo_args a = {};
    const at::Tensor& rewards = tensor(v[0]);
    if (!rewards.is_cuda()) throw Other();
    const int dev = rewards.get_device();
    const int64_t R = rewards.numel(), n = tensor(v[2]).numel();
    a.G = i32(v[4]);
    if (a.G <= 0 || R % a.G) throw Other();
    const int64_t ng = R / a.G;
    a.n_groups = size32(ng);
    a.n = size32(n);
    a.rewards = (const float*)ptr(v[0], kF, R, dev);
    a.offsets = (const int32_t*)ptr(v[1], kI, R + 1, dev);
    a.lp_new = (const float*)ptr(v[2], kF, n, dev);
    a.lp_old = (const float*)ptr(v[3], kF, n, dev);
    a.eps = f32(v[5]);
    a.out_group_obj = (float*)ptr(v[6], kF, ng, dev);
    a.out_skipped = (uint8_t*)ptr(v[7], kB, ng, dev);
    a.out_J = (float*)ptr(v[8], kF, 1, dev);
    a.out_adv = (float*)opt(v[9], kF, R, dev);
    a.out_ratio = (float*)opt(v[10], kF, n, dev);
    a.out_term = (float*)opt(v[11], kF, n, dev);
    a.out_rollout_obj = (float*)opt(v[12], kF, R, dev);
    a.stream = stream(v[13], dev);
    return call(g_grpo, a);
  });
}

PyObject* select(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 17, [&] {
    fork_select_args a = {};
    const at::Tensor& conf = tensor(v[0]);
    if (!conf.is_cuda()) throw Other();
    const int dev = conf.get_device();
    a.block_len = i32(v[5]);
    a.tau = f32(v[6]);
    a.B = i32(v[8]);
    a.L = i32(v[9]);
    const int64_t M = (int64_t)a.B * a.L;
    a.conf = (const float*)ptr(v[0], kF, M, dev);
    a.argmax = (const int32_t*)ptr(v[1], kI, M, dev);
    a.tokens = (int32_t*)ptr(v[2], kI, M, dev);
    a.mask = (uint8_t*)ptr(v[3], kB, M, dev);
    a.block_start = (int32_t*)ptr(v[4], kI, a.B, dev);
    a.out_fallback = (int32_t*)ptr(v[7], kI, a.B, dev);
    a.rule = i32(v[10]);
    a.entropy = (const float*)opt(v[11], kF, M, dev);
    a.uniform = (const float*)opt(v[12], kF, a.B, dev);
    a.out_ncommit = (int32_t*)opt(v[13], kI, a.B, dev);
    a.out_commit_pos = (int32_t*)opt(v[14], kI, (int64_t)a.B * a.block_len, dev);
    a.stream = stream(v[15], dev);
    a.layout = i32(v[16]);
    return call(g_select, a);
  });
}

PyObject* top_entropy(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 4, [&]() -> PyObject* {
    const at::Tensor& e = tensor(v[0]);
    if (e.dim() != 2 || !e.is_cuda()) throw Other();
    const int dev = e.get_device();
    const int32_t R = size32(e.size(0)), Lg = size32(e.size(1)), k = i32(v[1]);
    const float* in = (const float*)ptr(v[0], kF, (int64_t)R * Lg, dev);
    uint8_t* out = (uint8_t*)ptr(v[2], kB, (int64_t)R * Lg, dev);
    void* s = stream(v[3], dev);
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_top(in, R, Lg, k, out, s);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  });
}

// init(raw_stream, step_ex, step_noalloc, logprob, grpo, select, top_entropy):
// torch's raw-stream function and the addresses of the library's functions.
PyObject* init(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  if (nargs != 7) {
    PyErr_SetString(PyExc_TypeError, "init takes 7 arguments");
    return nullptr;
  }
  void* p[6];
  for (int i = 0; i < 6; ++i) {
    p[i] = PyLong_AsVoidPtr(v[i + 1]);
    if (!p[i]) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null function address");
      return nullptr;
    }
  }
  g_step_ex = (decltype(g_step_ex))p[0];
  g_step_noalloc = (decltype(g_step_noalloc))p[1];
  g_logprob = (decltype(g_logprob))p[2];
  g_grpo = (decltype(g_grpo))p[3];
  g_select = (decltype(g_select))p[4];
  g_top = (decltype(g_top))p[5];
  Py_INCREF(v[0]);
  Py_XSETREF(g_raw_stream, v[0]);
  Py_RETURN_NONE;
}

#define FORK_METHOD(NAME) {#NAME, (PyCFunction)(void (*)(void))NAME, METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {FORK_METHOD(init),   FORK_METHOD(step),        FORK_METHOD(logprob),
                          FORK_METHOD(grpo),   FORK_METHOD(select),      FORK_METHOD(top_entropy),
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_fastcall", nullptr, -1, kMethods};

}  // namespace

PyMODINIT_FUNC PyInit__fastcall(void) { return PyModule_Create(&kModule); }
