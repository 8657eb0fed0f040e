// The calls of the binding that a program makes again and again, marshalled in C++ (module _host): torq_linear,
// torq_rotate_quantize (and _fmt), torq_block_gram (and _positions) and torq_code_histogram.  The kernels of the smallest of
// them take 3 to 6 us, the interpreter 8 to 13 for the attribute look-ups, checks, allocations and a ctypes call.  One row
// through a 4096 x 4096 layer, a call among others: 10.2 us -> 5.6 or 6.4 from one process to the next (the kernel, replayed from a
// graph, 5.7).
//
// A function here takes a call only where everything about it is plain: exact tensors (no subclass), the shapes, types and
// layout that the library takes.  Anything else it leaves alone, returns None, and binding.py's own Python goes through the
// arguments one by one and raises what it always raised.  Same allocations, same C ABI, the status checked by the same
// function; no state but the addresses handed over in bind().
#include <Python.h>

#include <torch/csrc/Stream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <ATen/ATen.h>

#include <algorithm>
#include <cstdint>
#include <optional>

namespace {

using at::Tensor;

// the library's entry points and the binding's two functions
int (*f_linear)(const void *, const void *, const void *, const void *, void *, int64_t, int64_t, void *, size_t, void *);
size_t (*f_linear_bytes)(int64_t, int64_t, int);
int (*f_rotate_quantize)(const void *, const void *, int64_t, void *, void *, void *);
int (*f_rotate_quantize_fmt)(const void *, const void *, int64_t, int, float, void *, void *, void *);
int (*f_gram)(const void *, int64_t, int, int, void *, void *, size_t, void *);
int (*f_gram_positions)(const void *, int64_t, int, int, void *, void *, size_t, void *);
size_t (*f_gram_bytes)(int);
int (*f_histogram)(const void *, int64_t, int, void *, void *, size_t, void *);
size_t (*f_histogram_bytes)();
PyObject *py_stream, *py_check;
PyObject *s_handle, *s_value, *s_d;

struct NotPlain {};

const Tensor &tensor(PyObject *o) {
  if (!THPVariable_CheckExact(o)) throw NotPlain{};
  return THPVariable_Unpack(o);
}
void *address(const Tensor &t, at::ScalarType type) {
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) throw NotPlain{};
  return t.data_ptr();
}
int64_t integer(PyObject *o) {
  if (!PyLong_CheckExact(o)) throw NotPlain{};
  const int64_t v = PyLong_AsLongLong(o);
  if (v == -1 && PyErr_Occurred()) throw NotPlain{};
  return v;
}
int small_integer(PyObject *o) {
  const int64_t v = integer(o);
  if (v < 0 || v > 0x7FFFFFFF) throw NotPlain{};
  return (int)v;
}
struct Ref {
  PyObject *p;
  explicit Ref(PyObject *o) : p(o) {
    if (!p) throw NotPlain{};
  }
  ~Ref() { Py_DECREF(p); }
  Ref(const Ref &) = delete;
  Ref &operator=(const Ref &) = delete;
};
// an address held by a Python integer
void *pointer(PyObject *o) {
  if (!PyLong_Check(o)) throw NotPlain{};
  void *p = PyLong_AsVoidPtr(o);
  if (!p && PyErr_Occurred()) throw NotPlain{};
  return p;
}
// Rotation.handle, a ctypes pointer (None once it is closed)
void *handle_of(PyObject *rot) {
  Ref h(PyObject_GetAttr(rot, s_handle));
  if (h.p == Py_None) throw NotPlain{};
  Ref v(PyObject_GetAttr(h.p, s_value));
  return pointer(v.p);
}
int64_t d_of(PyObject *rot) {
  Ref d(PyObject_GetAttr(rot, s_d));
  return integer(d.p);
}
void *stream_of(PyObject *stream) {
  Ref s(PyObject_CallOneArg(py_stream, stream));
  return pointer(s.p);
}

// The stream of a call that allocates its own workspace: that goes back to the allocator when the call returns, ahead of the
// kernels that use it, so a stream that is not the one it is allocated on has to be known there.
std::optional<c10::Stream> user_of(PyObject *stream, const Tensor *workspace) {
  if (workspace || stream == Py_None) return std::nullopt;
  if (!THPStream_Check(stream)) throw NotPlain{};
  const THPStream *s = reinterpret_cast<const THPStream *>(stream);
  return c10::Stream::unpack3(s->stream_id, (c10::DeviceIndex)s->device_index, (c10::DeviceType)s->device_type);
}

// allocations and launches without the interpreter's lock, as ctypes and torch's own functions do them
struct Unlocked {
  PyThreadState *state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

Tensor given_or_new(const Tensor *given, const Tensor &like, at::IntArrayRef sizes, at::ScalarType type) {
  return given ? *given : like.new_empty(sizes, like.options().dtype(type));
}
Tensor scratch(const Tensor *given, const Tensor &like, int64_t bytes, const std::optional<c10::Stream> &user) {
  if (given) return *given;
  Tensor t = like.new_empty({bytes}, like.options().dtype(at::kByte));
  if (user) t.record_stream(*user);
  return t;
}
const Tensor *optional(PyObject *o) { return o == Py_None ? nullptr : &tensor(o); }
PyObject *wrapped(PyObject *given, const Tensor &t) {
  if (given == Py_None) return THPVariable_Wrap(t);
  Py_INCREF(given);
  return given;
}
// None of the arguments has been used if this returns nullptr without an error set
bool ok(int status, const char *what) {
  if (status == 0) return true;
  PyObject *r = PyObject_CallFunction(py_check, "is", status, what);
  Py_XDECREF(r);
  return false;
}

template <class F>
PyObject *plain_or_none(F &&f) {
  try {
    return f();
  } catch (...) {
    // (an interrupt that arrived while the interpreter was asked for something says nothing about the arguments)
    if (PyErr_Occurred() && !PyErr_ExceptionMatches(PyExc_Exception)) return nullptr;
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// linear(rot, x, W_q, W_s, out, workspace, stream)
PyObject *linear(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return plain_or_none([&]() -> PyObject * {
    if (n != 7) throw NotPlain{};
    const Tensor &x = tensor(a[1]), &W_q = tensor(a[2]), &W_s = tensor(a[3]);
    const Tensor *out_in = optional(a[4]), *ws_in = optional(a[5]);
    if (x.dim() != 2 || W_q.dim() != 2 || W_s.dim() != 2) throw NotPlain{};
    const int64_t M = x.size(0), d = x.size(1), N = W_q.size(0);
    if (d != d_of(a[0]) || W_q.size(1) != d / 2 || W_s.size(0) != N || W_s.size(1) != d / 32) throw NotPlain{};
    void *const handle = handle_of(a[0]), *const xp = address(x, at::kBFloat16), *const qp = address(W_q, at::kByte),
                *const sp = address(W_s, at::kByte), *const stream = stream_of(a[6]);
    const std::optional<c10::Stream> user = user_of(a[6], ws_in);
    Tensor out;
    int status;
    {
      Unlocked unlocked;
      const Tensor ws = scratch(ws_in, x, ws_in ? 1 : std::max<int64_t>((int64_t)f_linear_bytes(M, N, (int)d), 1), user);
      out = given_or_new(out_in, x, {M, N}, at::kBFloat16);
      status = f_linear(handle, xp, qp, sp, address(out, at::kBFloat16), M, N, address(ws, at::kByte), (size_t)ws.numel(), stream);
    }
    return ok(status, "torq_linear") ? wrapped(a[4], out) : nullptr;
  });
}

// rotate_quantize(rot, x, format or None, global_scale, codes, scales, stream)
PyObject *rotate_quantize(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return plain_or_none([&]() -> PyObject * {
    if (n != 7) throw NotPlain{};
    const Tensor &x = tensor(a[1]);
    const Tensor *codes_in = optional(a[4]), *scales_in = optional(a[5]);
    const bool with_format = a[2] != Py_None;
    const int format = with_format ? small_integer(a[2]) : 0;
    if (!PyFloat_CheckExact(a[3]) || x.dim() != 2) throw NotPlain{};
    const float global_scale = (float)PyFloat_AS_DOUBLE(a[3]);
    const int64_t M = x.size(0), d = x.size(1);
    if (d != d_of(a[0])) throw NotPlain{};
    void *const handle = handle_of(a[0]), *const xp = address(x, at::kBFloat16), *const stream = stream_of(a[6]);
    Tensor codes, scales;
    int status;
    {
      Unlocked unlocked;
      codes = given_or_new(codes_in, x, {M, d / 2}, at::kByte);
      scales = given_or_new(scales_in, x, {M, format == 2 ? d / 16 : d / 32}, at::kByte);
      void *const cp = address(codes, at::kByte), *const sp = address(scales, at::kByte);
      status = with_format ? f_rotate_quantize_fmt(handle, xp, M, format, global_scale, cp, sp, stream)
                           : f_rotate_quantize(handle, xp, M, cp, sp, stream);
    }
    if (!ok(status, with_format ? "torq_rotate_quantize_fmt" : "torq_rotate_quantize")) return nullptr;
    PyObject *c = wrapped(a[4], codes), *s = wrapped(a[5], scales), *pair = c && s ? PyTuple_Pack(2, c, s) : nullptr;
    Py_XDECREF(c);
    Py_XDECREF(s);
    return pair;
  });
}

// gram(x, G, positions, Sigma, workspace, stream)
PyObject *gram(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return plain_or_none([&]() -> PyObject * {
    if (n != 6) throw NotPlain{};
    const Tensor &x = tensor(a[0]);
    const Tensor *sigma_in = optional(a[3]), *ws_in = optional(a[4]);
    const int G = small_integer(a[1]);
    const bool positions = a[2] == Py_True;
    if (x.dim() != 2 || x.size(1) > 0x7FFFFFFF) throw NotPlain{};
    const int64_t M = x.size(0), d = x.size(1);
    void *const xp = address(x, at::kBFloat16), *const stream = stream_of(a[5]);
    const std::optional<c10::Stream> user = user_of(a[5], ws_in);
    Tensor sigma;
    int status;
    {
      Unlocked unlocked;
      const int64_t shape[3] = {32, G, G};
      sigma = given_or_new(sigma_in, x, positions ? at::IntArrayRef(shape, 3) : at::IntArrayRef(shape + 1, 2), at::kDouble);
      const Tensor ws = scratch(ws_in, x, ws_in ? 1 : std::max<int64_t>((int64_t)f_gram_bytes(G), 16), user);
      status = (positions ? f_gram_positions : f_gram)(xp, M, (int)d, G, address(sigma, at::kDouble), address(ws, at::kByte),
                                                       (size_t)ws.numel(), stream);
    }
    return ok(status, positions ? "torq_block_gram_positions" : "torq_block_gram") ? wrapped(a[3], sigma) : nullptr;
  });
}

// histogram(codes, d, counts, workspace, stream)
PyObject *histogram(PyObject *, PyObject *const *a, Py_ssize_t n) {
  return plain_or_none([&]() -> PyObject * {
    if (n != 5) throw NotPlain{};
    const Tensor &codes = tensor(a[0]);
    const Tensor *counts_in = optional(a[2]), *ws_in = optional(a[3]);
    const int d = small_integer(a[1]);
    if (codes.dim() != 2 || codes.size(1) * 2 != d) throw NotPlain{};
    void *const cp = address(codes, at::kByte), *const stream = stream_of(a[4]);
    const std::optional<c10::Stream> user = user_of(a[4], ws_in);
    Tensor counts;
    int status;
    {
      Unlocked unlocked;
      counts = given_or_new(counts_in, codes, {32, 8}, at::kLong);
      const Tensor ws = scratch(ws_in, codes, ws_in ? 1 : (int64_t)f_histogram_bytes(), user);
      status = f_histogram(cp, codes.size(0), d, address(counts, at::kLong), address(ws, at::kByte), (size_t)ws.numel(), stream);
    }
    return ok(status, "torq_code_histogram") ? wrapped(a[2], counts) : nullptr;
  });
}

// bind({entry point: address}, stream function, check function)
PyObject *bind(PyObject *, PyObject *args) {
  PyObject *entries, *stream, *check;
  if (!PyArg_ParseTuple(args, "O!OO", &PyDict_Type, &entries, &stream, &check)) return nullptr;
#define TORQ_BIND(VAR_, NAME_)                                                                    \
  {                                                                                               \
    PyObject *v = PyDict_GetItemString(entries, NAME_);                                           \
    void *p = v ? PyLong_AsVoidPtr(v) : nullptr;                                                  \
    if (!p) return PyErr_Occurred() ? nullptr : PyErr_Format(PyExc_KeyError, "%s", NAME_);        \
    VAR_ = reinterpret_cast<decltype(VAR_)>(p);                                                   \
  }
  TORQ_BIND(f_linear, "torq_linear")
  TORQ_BIND(f_linear_bytes, "torq_linear_workspace_bytes_n")
  TORQ_BIND(f_rotate_quantize, "torq_rotate_quantize")
  TORQ_BIND(f_rotate_quantize_fmt, "torq_rotate_quantize_fmt")
  TORQ_BIND(f_gram, "torq_block_gram")
  TORQ_BIND(f_gram_positions, "torq_block_gram_positions")
  TORQ_BIND(f_gram_bytes, "torq_block_gram_workspace_bytes")
  TORQ_BIND(f_histogram, "torq_code_histogram")
  TORQ_BIND(f_histogram_bytes, "torq_code_histogram_workspace_bytes")
#undef TORQ_BIND
  Py_INCREF(stream);
  Py_INCREF(check);
  Py_XDECREF(py_stream);
  Py_XDECREF(py_check);
  py_stream = stream;
  py_check = check;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"bind", bind, METH_VARARGS, nullptr},
    {"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(linear)), METH_FASTCALL, nullptr},
    {"rotate_quantize", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(rotate_quantize)), METH_FASTCALL, nullptr},
    {"gram", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(gram)), METH_FASTCALL, nullptr},
    {"histogram", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(histogram)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() {
  s_handle = PyUnicode_InternFromString("handle");
  s_value = PyUnicode_InternFromString("value");
  s_d = PyUnicode_InternFromString("d");
  if (!s_handle || !s_value || !s_d) return nullptr;
  PyObject *m = PyModule_Create(&module);
  // (binding.py binds no module built against another torch)
  if (m && PyModule_AddStringConstant(m, "torch_version", TORQ_TORCH_VERSION) != 0) Py_CLEAR(m);
  return m;
}
