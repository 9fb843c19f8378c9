// The Python binding's way of a good call, in native code: the arguments are checked and handed to the C entry point
// without an interpreter step per tensor (CPython extension module `_args`, used by binding.py).
//
// A call of a decode step passes some ten tensors, each with three or four attribute look-ups from Python, and fifteen
// values through ctypes.  One copris_is_ratio of ten tensors took 7.2 us of a host thread and takes 4.0, of which its
// launch is 3.1; a decode step of five such calls over two requests, where the host is the slower side, went from 38.4
// to 26.6 us.
//
// Every function takes the arguments of the binding's function of that name in order, `stream` last, and returns the
// entry point's code, or None if anything about the arguments is not the plain case: not a torch.Tensor itself, on the
// CPU, not contiguous, of another type or rank, a stream object, a number of another type or out of range.  Nothing has
// been called then, and the binding goes through its own checks, which name the argument.  Nothing is kept from a call.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cxxabi.h>

#include <optional>
#include <tuple>

#include <torch/csrc/autograd/python_variable.h>

#include "copris.h"

namespace {

// the entry points of the library that the binding has loaded, in the order of kNames
enum Entry { kApply, kAppend, kTrajAppend, kGather, kDecode, kPrefill, kSample, kGiven, kRatio, kSurrogate, kEntries };
const char* const kNames[kEntries] = {"copris_rollout_apply", "copris_kv_append", "copris_traj_append",
                                      "copris_traj_gather", "copris_decode_attn", "copris_prefill_attn",
                                      "copris_lmhead_logprob", "copris_lmhead_token_logprob", "copris_is_ratio",
                                      "copris_grpo_surrogate"};
void* g_entry[kEntries] = {};
PyObject* g_raw_stream = nullptr;   // device index -> raw handle of torch's current stream

struct Plain {};                    // thrown where the plain case ends

// The arguments of one call.
struct Args {
  PyObject* const* v;
  Py_ssize_t n;

  const at::Tensor& tensor(int i) const {
    if (!THPVariable_CheckExact(v[i])) throw Plain();
    const at::Tensor& t = THPVariable_Unpack(v[i]);
    if (!t.is_cuda() || !t.is_contiguous()) throw Plain();
    return t;
  }
  template <typename T = void> T* data(int i) const { return static_cast<T*>(tensor(i).data_ptr()); }
  template <typename T = void> T* data(int i, at::ScalarType type) const {
    const at::Tensor& t = tensor(i);
    if (t.scalar_type() != type) throw Plain();
    return static_cast<T*>(t.data_ptr());
  }
  template <typename T> T* optional(int i, at::ScalarType type) const {
    return v[i] == Py_None ? nullptr : data<T>(i, type);
  }
  float* f32(int i) const { return data<float>(i, at::kFloat); }
  int32_t* i32(int i) const { return data<int32_t>(i, at::kInt); }
  int64_t* i64(int i) const { return data<int64_t>(i, at::kLong); }
  int64_t size(int i, int d, int dims) const {
    const at::Tensor& t = tensor(i);
    if (t.dim() != dims) throw Plain();
    return t.size(d);
  }
  int size32(int i, int d, int dims) const { return narrow(size(i, d, dims)); }
  int64_t numel(int i) const { return tensor(i).numel(); }
  static int narrow(int64_t x) {
    if (x < INT32_MIN || x > INT32_MAX) throw Plain();
    return static_cast<int>(x);
  }
  int integer(int i) const {
    if (!PyLong_CheckExact(v[i])) throw Plain();
    int overflow = 0;
    const long long x = PyLong_AsLongLongAndOverflow(v[i], &overflow);
    if (overflow != 0) throw Plain();
    return narrow(x);
  }
  uint64_t seed(int i) const {
    if (!PyLong_CheckExact(v[i])) throw Plain();
    return PyLong_AsUnsignedLongLongMask(v[i]);
  }
  float number(int i) const {
    if (!PyFloat_CheckExact(v[i])) throw Plain();
    return static_cast<float>(PyFloat_AS_DOUBLE(v[i]));
  }
  at::ScalarType element(int i) const {
    const int code = integer(i);
    if (code != COPRIS_BF16 && code != COPRIS_F32) throw Plain();
    return code == COPRIS_BF16 ? at::kBFloat16 : at::kFloat;
  }
  // the current stream of the device that argument `ref` lives on (the last argument has to be None)
  void* stream(int ref) const {
    if (v[n - 1] != Py_None) throw Plain();
    PyObject* dev = PyLong_FromLong(tensor(ref).get_device());
    PyObject* h = dev ? PyObject_CallOneArg(g_raw_stream, dev) : nullptr;
    Py_XDECREF(dev);
    if (!h) throw Plain();
    void* p = PyLong_AsVoidPtr(h);
    Py_DECREF(h);
    if (PyErr_Occurred()) throw Plain();
    return p;
  }
};

// The checked arguments of one entry point, as it takes them.
template <typename F> struct Ready;
template <typename... P> struct Ready<int(P...)> {
  Entry entry;
  std::tuple<P...> values;
  int operator()() const { return std::apply(reinterpret_cast<int (*)(P...)>(g_entry[entry]), values); }
};
#define READY(e, f, ...) Ready<decltype(f)>{e, {__VA_ARGS__}}

auto rollout_apply(const Args& a) {
  return READY(kApply, copris_rollout_apply, a.i32(0), a.integer(1), a.integer(2), a.i64(3), a.i32(4), a.i32(5),
               a.i32(6), a.size32(6, 0, 2), a.size32(6, 1, 2), a.stream(6));
}
auto kv_append(const Args& a) {
  return READY(kAppend, copris_kv_append, a.data(0), a.data(1), a.i32(2), a.i32(3), a.data(4), a.data(5),
               a.size32(0, 0, 3), a.size32(0, 1, 3), a.size32(0, 2, 3), a.size32(4, 2, 4), a.size32(2, 1, 2),
               a.size(4, 0, 4), a.integer(6), a.stream(4));
}
auto traj_append(const Args& a) {
  return READY(kTrajAppend, copris_traj_append, a.i32(0), a.f32(1), a.i64(2), a.i32(3), a.i32(4), a.integer(5),
               a.i32(6), a.f32(7), a.i32(8), Args::narrow(a.numel(0)), a.size(6, 0, 2), a.size32(6, 1, 2),
               a.stream(6));
}
auto traj_gather(const Args& a) {
  return READY(kGather, copris_traj_gather, a.i32(0), a.f32(1), a.i32(2), a.i32(3), a.i32(4), a.integer(5), a.i32(6),
               a.f32(7), a.f32(8), a.i32(9), Args::narrow(a.numel(3)), a.size(0, 0, 2), a.size32(0, 1, 2),
               a.stream(0));
}
auto decode_attn(const Args& a) {   // ..., workspace, scale, dtype, stream
  const at::ScalarType e = a.element(9);
  return READY(kDecode, copris_decode_attn, a.data(0, e), a.data(1, e), a.data(2, e), a.i32(3), a.i32(4),
               a.data(5, e), a.optional<float>(6, at::kFloat), a.data(7, at::kByte), a.numel(7), a.size32(0, 0, 3),
               a.size32(0, 1, 3), a.size32(1, 1, 4), a.size32(0, 2, 3), a.size32(1, 2, 4), a.size32(3, 1, 2),
               a.size(1, 0, 4), a.number(8), a.integer(9), a.stream(0));
}
auto prefill_attn(const Args& a) {   // ..., lse, max_seqlen, scale, dtype, stream
  const at::ScalarType e = a.element(11);
  return READY(kPrefill, copris_prefill_attn, a.data(0, e), a.data(1, e), a.data(2, e), a.i32(3), a.i32(4),
               a.data(5, e), a.data(6, e), a.data(7, e), a.optional<float>(8, at::kFloat),
               Args::narrow(a.numel(3) - 1), a.size(0, 0, 3), a.size32(0, 1, 3), a.size32(1, 1, 3),
               a.size32(0, 2, 3), a.size32(5, 2, 4), a.size32(4, 1, 2), a.size(5, 0, 4), a.integer(9), a.number(10),
               a.integer(11), a.stream(0));
}
auto lmhead_logprob(const Args& a) {   // ..., workspace, seed, temperature, dtype, stream
  const at::ScalarType e = a.element(10);
  return READY(kSample, copris_lmhead_logprob, a.data(0, e), a.data(1, e), a.i64(2), a.i32(3), a.seed(8),
               a.number(9), a.i32(4), a.f32(5), a.optional<float>(6, at::kFloat), a.data(7, at::kByte), a.numel(7),
               a.size32(0, 0, 2), a.size32(0, 1, 2), a.size32(1, 0, 2), a.integer(10), a.stream(0));
}
auto lmhead_token_logprob(const Args& a) {   // ..., workspace, temperature, dtype, stream
  const at::ScalarType e = a.element(7);
  return READY(kGiven, copris_lmhead_token_logprob, a.data(0, e), a.data(1, e), a.i32(2), a.number(6), a.f32(3),
               a.optional<float>(4, at::kFloat), a.data(5, at::kByte), a.numel(5), a.size32(0, 0, 2),
               a.size32(0, 1, 2), a.size32(1, 0, 2), a.integer(7), a.stream(0));
}
auto is_ratio(const Args& a) {   // ..., seq_nclip, eps_low, eps_high, stream
  return READY(kRatio, copris_is_ratio, a.f32(0), a.f32(1), a.f32(2), a.i32(3), a.i32(4),
               a.optional<uint8_t>(5, at::kByte), a.number(11), a.number(12), a.f32(6), a.f32(7), a.f32(8), a.i32(9),
               a.i32(10), Args::narrow(a.numel(3) - 1), a.numel(0), a.stream(3));
}
auto grpo_surrogate(const Args& a) {   // ..., objective, eps_low, eps_high, stream
  return READY(kSurrogate, copris_grpo_surrogate, a.f32(0), a.f32(1), a.f32(2), a.i32(3), a.i32(4),
               a.optional<uint8_t>(5, at::kByte), a.f32(6), a.number(12), a.number(13), a.f32(7), a.f32(8), a.f32(9),
               a.i32(10), a.f32(11), Args::narrow(a.numel(3) - 1), a.numel(0), a.stream(11));
}

// The call itself is made with the interpreter's lock given up, as ctypes does: a launch can wait for room in the queue.
// Asking for the lock again, Python ends a daemon's thread if the interpreter is ending, by unwinding its stack: no frame
// from here on is noexcept or catches that.
template <auto PREPARE, Py_ssize_t N>
PyObject* call(PyObject*, PyObject* const* v, Py_ssize_t n) {
  if (n != N || g_raw_stream == nullptr) Py_RETURN_NONE;
  std::optional<decltype(PREPARE(Args{v, n}))> ready;
  try {
    ready.emplace(PREPARE(Args{v, n}));
  } catch (abi::__forced_unwind&) {   // (the stream's look-up may run Python code)
    throw;
  } catch (...) {   // (no exception of torch's leaves this module either)
    PyErr_Clear();
    Py_RETURN_NONE;
  }
  PyThreadState* state = PyEval_SaveThread();
  const int code = (*ready)();        // (a C entry point throws nothing)
  PyEval_RestoreThread(state);
  return PyLong_FromLong(code);
}

// bind(addresses of kNames, raw_stream)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *addresses, *raw;
  if (!PyArg_ParseTuple(args, "O!O", &PyTuple_Type, &addresses, &raw)) return nullptr;
  if (PyTuple_GET_SIZE(addresses) != kEntries) {
    PyErr_SetString(PyExc_ValueError, "one address per entry point");
    return nullptr;
  }
  void* p[kEntries];
  for (int i = 0; i < kEntries; ++i) {
    p[i] = PyLong_AsVoidPtr(PyTuple_GET_ITEM(addresses, i));
    if (p[i] == nullptr) {
      if (!PyErr_Occurred()) PyErr_SetString(PyExc_ValueError, "null address");
      return nullptr;
    }
  }
  for (int i = 0; i < kEntries; ++i) g_entry[i] = p[i];
  Py_INCREF(raw);
  Py_XSETREF(g_raw_stream, raw);
  Py_RETURN_NONE;
}

#define FAST(name, n) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(&call<name, n>)), METH_FASTCALL, nullptr}
PyMethodDef kMethods[] = {FAST(rollout_apply, 8), FAST(kv_append, 8), FAST(traj_append, 10), FAST(traj_gather, 11),
                          FAST(decode_attn, 11), FAST(prefill_attn, 13), FAST(lmhead_logprob, 12),
                          FAST(lmhead_token_logprob, 9), FAST(is_ratio, 14), FAST(grpo_surrogate, 15), {"bind", bind, METH_VARARGS, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_args", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__args(void) {
  PyObject* m = PyModule_Create(&kModule);
  if (!m) return nullptr;
  PyObject* names = PyTuple_New(kEntries);
  if (!names) return nullptr;
  for (int i = 0; i < kEntries; ++i) PyTuple_SET_ITEM(names, i, PyUnicode_FromString(kNames[i]));
  if (PyModule_AddObject(m, "entry_points", names) != 0) return nullptr;
  // a tensor is read by its C++ layout, which is that of one PyTorch version
  if (PyModule_AddStringConstant(m, "built_for", COPRIS_TORCH_VERSION) != 0) return nullptr;
  return m;
}
