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

// Reads the arguments of one call.  An argument that the plain path does not
// take clears `ok`; what is read after that is of no use, and the call is not
// made.  It is not an exception because the first one thrown in a process has
// the unwinder read the tables of every library that torch has loaded: 84 ms.
struct Reader {
  bool ok = true;

  bool need(bool cond) {
    if (!cond) ok = false;
    return ok;
  }

  // Null for anything but a plain torch.Tensor.
  const at::Tensor* tensor(PyObject* o) {
    return need(THPVariable_CheckExact(o)) ? &THPVariable_Unpack(o) : nullptr;
  }

  // Device pointer of a contiguous tensor of `n` elements on device `dev`.
  void* ptr(PyObject* o, at::ScalarType type, int64_t n, int dev) {
    const at::Tensor* t = tensor(o);
    if (!t || !need(t->is_cuda() && t->get_device() == dev && t->scalar_type() == type &&
                    t->numel() == n && t->is_contiguous()))
      return nullptr;
    return t->data_ptr();
  }

  void* opt(PyObject* o, at::ScalarType type, int64_t n, int dev) {
    return o == Py_None ? nullptr : ptr(o, type, n, dev);
  }

  int64_t numel(PyObject* o) {
    const at::Tensor* t = tensor(o);
    return t ? t->numel() : 0;
  }

  // The device of a tensor that has to be on the GPU.
  int device(PyObject* o) {
    const at::Tensor* t = tensor(o);
    return t && need(t->is_cuda()) ? t->get_device() : -1;
  }

  // Sizes of a matrix; zeros for anything else.
  void sizes(PyObject* o, int64_t* rows, int64_t* cols) {
    const at::Tensor* t = tensor(o);
    const bool m = t && need(t->dim() == 2);
    *rows = m ? t->size(0) : 0;
    *cols = m ? t->size(1) : 0;
  }

  at::ScalarType type(PyObject* o) {
    const at::Tensor* t = tensor(o);
    return t ? t->scalar_type() : at::ScalarType::Undefined;
  }

  int32_t dtype(at::ScalarType t) {
    need(t == at::ScalarType::BFloat16 || t == at::ScalarType::Float);
    return t == at::ScalarType::BFloat16 ? FORK_BF16 : FORK_F32;
  }

  int32_t i32(PyObject* o) {
    if (!need(PyLong_CheckExact(o))) return 0;
    int overflow = 0;
    const long long v = PyLong_AsLongLongAndOverflow(o, &overflow);
    return need(!overflow && v >= INT32_MIN && v <= INT32_MAX) ? (int32_t)v : 0;
  }

  int32_t size32(int64_t v) { return need(v <= INT32_MAX) ? (int32_t)v : 0; }

  float f32(PyObject* o) {
    return need(PyFloat_CheckExact(o)) ? (float)PyFloat_AS_DOUBLE(o) : 0.f;
  }

  uint64_t bits(PyObject* o) {
    return need(PyLong_CheckExact(o)) ? PyLong_AsUnsignedLongLongMask(o) : 0;
  }

  void* handle(PyObject* o) {
    if (!need(o && PyLong_CheckExact(o))) return nullptr;
    void* p = PyLong_AsVoidPtr(o);
    if (!need(!PyErr_Occurred())) PyErr_Clear();
    return p;
  }

  // The given stream's handle, or the device's current stream's.
  void* stream(PyObject* s, int dev) {
    if (!ok) return nullptr;
    PyObject* v;
    if (s == Py_None) {
      PyObject* d = PyLong_FromLong(dev);
      v = d ? PyObject_CallFunctionObjArgs(g_raw_stream, d, nullptr) : nullptr;
      Py_XDECREF(d);
    } else {
      v = PyObject_GetAttrString(s, "cuda_stream");
    }
    if (!v) PyErr_Clear();
    void* p = handle(v);
    Py_XDECREF(v);
    return p;
  }

  // The pair of events around the LM-head kernel.
  void events(PyObject* o, void** begin, void** end) {
    if (o == Py_None || !need(PyTuple_CheckExact(o) && PyTuple_GET_SIZE(o) == 2)) return;
    *begin = handle(PyTuple_GET_ITEM(o, 0));
    *end = handle(PyTuple_GET_ITEM(o, 1));
  }

  void workspace(PyObject* o, int dev, void** p, size_t* n) {
    if (o == Py_None) return;
    const at::Tensor* t = tensor(o);
    if (!t || !need(t->is_cuda() && t->get_device() == dev && t->is_contiguous())) return;
    *p = t->data_ptr();
    *n = (size_t)t->numel() * t->element_size();
  }
};

constexpr auto kF = at::ScalarType::Float;
constexpr auto kI = at::ScalarType::Int;
constexpr auto kB = at::ScalarType::Byte;

template <class F, class A>
PyObject* call(F fn, const A& a) {
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(&a);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
}

// Runs `f` on a reader; None for what the plain path does not take.
template <class F>
PyObject* plain(Py_ssize_t n, Py_ssize_t want, F&& f) {
  if (n != want) {
    PyErr_Format(PyExc_TypeError, "expected %zd arguments, got %zd", want, n);
    return nullptr;
  }
  try {
    Reader r;
    if (PyObject* rc = f(r)) return rc;
    if (PyErr_Occurred()) return nullptr;
  } catch (...) {
    // a tensor without storage of its own
  }
  Py_RETURN_NONE;
}

PyObject* step(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 27, [&](Reader& r) -> PyObject* {
    fork_step_args a = {};
    const int dev = r.device(v[1]);
    int64_t M, d, V, dw;
    r.sizes(v[1], &M, &d);
    r.sizes(v[2], &V, &dw);
    const at::ScalarType type = r.type(v[1]);
    a.block_len = r.i32(v[6]);
    a.B = r.i32(v[12]);
    a.L = r.i32(v[13]);
    r.need(M == (int64_t)a.B * a.L);
    a.d = r.size32(d);
    a.V = r.size32(V);
    a.dtype = r.dtype(type);
    a.hidden = r.ptr(v[1], type, M * d, dev);
    a.W_head = r.ptr(v[2], type, V * d, dev);
    a.tokens = (int32_t*)r.ptr(v[3], kI, M, dev);
    a.mask = (uint8_t*)r.ptr(v[4], kB, M, dev);
    a.block_start = (int32_t*)r.ptr(v[5], kI, a.B, dev);
    a.tau = r.f32(v[7]);
    a.out_conf = (float*)r.ptr(v[8], kF, M, dev);
    a.out_entropy = (float*)r.ptr(v[9], kF, M, dev);
    a.out_logp = (float*)r.ptr(v[10], kF, M, dev);
    a.out_fallback = (int32_t*)r.ptr(v[11], kI, a.B, dev);
    a.out_lse = (float*)r.opt(v[14], kF, M, dev);
    a.out_argmax = (int32_t*)r.opt(v[15], kI, M, dev);
    a.out_ncommit = (int32_t*)r.opt(v[16], kI, a.B, dev);
    a.out_commit_pos = (int32_t*)r.opt(v[17], kI, (int64_t)a.B * a.block_len, dev);
    a.rule = r.i32(v[18]);
    r.workspace(v[19], dev, &a.workspace, &a.workspace_bytes);
    a.stream = r.stream(v[20], dev);
    r.events(v[21], &a.ev_lmhead_begin, &a.ev_lmhead_end);
    a.fallback_uniform = (const float*)r.opt(v[22], kF, a.B, dev);
    a.rows_mode = r.i32(v[23]);
    a.sample_temperature = r.f32(v[24]);
    a.sample_seed = r.bits(v[25]);
    a.sample_counter = (uint32_t)r.bits(v[26]);
    return r.ok ? call(v[0] == Py_True ? g_step_noalloc : g_step_ex, a) : nullptr;
  });
}

PyObject* logprob(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 11, [&](Reader& r) -> PyObject* {
    fork_logprob_args a = {};
    const int dev = r.device(v[0]);
    int64_t M, d, V, dw;
    r.sizes(v[0], &M, &d);
    r.sizes(v[1], &V, &dw);
    const int64_t n = r.numel(v[2]);
    const at::ScalarType type = r.type(v[0]);
    a.n = r.size32(n);
    a.M = r.size32(M);
    a.d = r.size32(d);
    a.V = r.size32(V);
    a.dtype = r.dtype(type);
    a.hidden = r.ptr(v[0], type, M * d, dev);
    a.W_head = r.ptr(v[1], type, V * d, dev);
    a.tokens = (const int32_t*)r.ptr(v[2], kI, n, dev);
    a.out_logp = (float*)r.ptr(v[3], kF, n, dev);
    a.rows = (const int32_t*)r.opt(v[4], kI, n, dev);
    a.out_q = (float*)r.opt(v[5], kF, n, dev);
    a.out_entropy = (float*)r.opt(v[6], kF, n, dev);
    a.out_lse = (float*)r.opt(v[7], kF, n, dev);
    r.need(v[8] == Py_None);  // a caller workspace is not checked here
    a.stream = r.stream(v[9], dev);
    r.events(v[10], &a.ev_lmhead_begin, &a.ev_lmhead_end);
    return r.ok ? call(g_logprob, a) : nullptr;
  });
}

PyObject* grpo(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 14, [&](Reader& r) -> PyObject* {
    fork_grpo_args a = {};
    const int dev = r.device(v[0]);
    const int64_t R = r.numel(v[0]), n = r.numel(v[2]);
    a.G = r.i32(v[4]);
    if (!r.need(a.G > 0 && R % a.G == 0)) return nullptr;
    const int64_t ng = R / a.G;
    a.n_groups = r.size32(ng);
    a.n = r.size32(n);
    a.rewards = (const float*)r.ptr(v[0], kF, R, dev);
    a.offsets = (const int32_t*)r.ptr(v[1], kI, R + 1, dev);
    a.lp_new = (const float*)r.ptr(v[2], kF, n, dev);
    a.lp_old = (const float*)r.ptr(v[3], kF, n, dev);
    a.eps = r.f32(v[5]);
    a.out_group_obj = (float*)r.ptr(v[6], kF, ng, dev);
    a.out_skipped = (uint8_t*)r.ptr(v[7], kB, ng, dev);
    a.out_J = (float*)r.ptr(v[8], kF, 1, dev);
    a.out_adv = (float*)r.opt(v[9], kF, R, dev);
    a.out_ratio = (float*)r.opt(v[10], kF, n, dev);
    a.out_term = (float*)r.opt(v[11], kF, n, dev);
    a.out_rollout_obj = (float*)r.opt(v[12], kF, R, dev);
    a.stream = r.stream(v[13], dev);
    return r.ok ? call(g_grpo, a) : nullptr;
  });
}

PyObject* select(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 17, [&](Reader& r) -> PyObject* {
    fork_select_args a = {};
    const int dev = r.device(v[0]);
    a.block_len = r.i32(v[5]);
    a.tau = r.f32(v[6]);
    a.B = r.i32(v[8]);
    a.L = r.i32(v[9]);
    const int64_t M = (int64_t)a.B * a.L;
    a.conf = (const float*)r.ptr(v[0], kF, M, dev);
    a.argmax = (const int32_t*)r.ptr(v[1], kI, M, dev);
    a.tokens = (int32_t*)r.ptr(v[2], kI, M, dev);
    a.mask = (uint8_t*)r.ptr(v[3], kB, M, dev);
    a.block_start = (int32_t*)r.ptr(v[4], kI, a.B, dev);
    a.out_fallback = (int32_t*)r.ptr(v[7], kI, a.B, dev);
    a.rule = r.i32(v[10]);
    a.entropy = (const float*)r.opt(v[11], kF, M, dev);
    a.uniform = (const float*)r.opt(v[12], kF, a.B, dev);
    a.out_ncommit = (int32_t*)r.opt(v[13], kI, a.B, dev);
    a.out_commit_pos = (int32_t*)r.opt(v[14], kI, (int64_t)a.B * a.block_len, dev);
    a.stream = r.stream(v[15], dev);
    a.layout = r.i32(v[16]);
    return r.ok ? call(g_select, a) : nullptr;
  });
}

PyObject* top_entropy(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  return plain(nargs, 4, [&](Reader& r) -> PyObject* {
    const int dev = r.device(v[0]);
    int64_t rows, cols;
    r.sizes(v[0], &rows, &cols);
    const int32_t R = r.size32(rows), Lg = r.size32(cols), k = r.i32(v[1]);
    const float* in = (const float*)r.ptr(v[0], kF, (int64_t)R * Lg, dev);
    uint8_t* out = (uint8_t*)r.ptr(v[2], kB, (int64_t)R * Lg, dev);
    void* s = r.stream(v[3], dev);
    if (!r.ok) return nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = g_top(in, R, Lg, k, out, s);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(rc);
  });
}

// init(raw_stream, sizes of the four argument structures, step_ex,
// step_noalloc, logprob, grpo, select, top_entropy): torch's raw-stream
// function, what the caller takes the structures to be, and the addresses of
// the library's functions.
PyObject* init(PyObject*, PyObject* const* v, Py_ssize_t nargs) {
  if (nargs != 11) {
    PyErr_SetString(PyExc_TypeError, "init takes 11 arguments");
    return nullptr;
  }
  const size_t sizes[4] = {sizeof(fork_step_args), sizeof(fork_logprob_args),
                           sizeof(fork_grpo_args), sizeof(fork_select_args)};
  for (int i = 0; i < 4; ++i) {
    const size_t n = PyLong_AsSize_t(v[i + 1]);
    if (PyErr_Occurred()) return nullptr;
    if (n != sizes[i]) {
      PyErr_SetString(PyExc_ImportError, "built for other argument structures");
      return nullptr;
    }
  }
  void* p[6];
  for (int i = 0; i < 6; ++i) {
    p[i] = PyLong_AsVoidPtr(v[i + 5]);
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
