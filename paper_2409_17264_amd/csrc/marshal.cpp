// Argument marshalling of the Python binding's tensor calls: what binding.py does with a call's
// arguments, in native code.  An ordinary call (plain tensors, lengths as int32 or int64 arrays or as
// lists of integers, everything in order) is made from here; every other one is answered with None,
// with nothing enqueued, and binding.py then goes through it step by step, converts what can be
// converted and raises what has to be raised.  Only an error of the HIP runtime, with which some of a
// call may be enqueued, is raised from here, and the call not made again.  (Host time of one decode at
// 2048 tokens, its append and its attention: 23.9 us in Python, of which 7 us were the three launches
// and 5 us the three allocations; 12 us from here.)
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <ATen/ATen.h>
#include <c10/util/SmallVector.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <algorithm>
#include <cstdint>
#include <cstring>
#include <exception>
#include <limits>
#include <type_traits>

#include "medha.h"
#include "medha_internal.h"

namespace {

// Entry points of libmedha.so (bind()), and the binding's functions for torch's current stream and
// for error codes.
struct Library {
  decltype(&medha_chunked_prefill_attn) prefill = nullptr;
  decltype(&medha_chunked_prefill_attn_alloc) prefill_alloc = nullptr;
  decltype(&medha_decode_partial_attn) decode = nullptr;
  decltype(&medha_decode_partial_workspace_bytes) decode_bytes = nullptr;
  decltype(&medha_chunk_partial_attn) chunk = nullptr;
  decltype(&medha_chunk_partial_workspace_bytes) chunk_bytes = nullptr;
  decltype(&medha_lse_merge) merge = nullptr;
  decltype(&medha_kv_append) append = nullptr;
  PyObject* stream = nullptr;
  PyObject* check = nullptr;  // raises an error code of the library's
} lib;

// A host array of the caller's, copied: the call runs without the interpreter's lock.
template <class T>
class HostArray {
 public:
  // Takes C-contiguous buffers of int32 and int64 and lists and tuples of Python's integers, as long
  // as T holds their values; false for anything else.  (The arrays are a call's first checks: what
  // has to go the long way is most often found here, and costs least to find out.)
  bool take(PyObject* o) {
    if (PyList_CheckExact(o) || PyTuple_CheckExact(o)) return take_sequence(o);
    if (!PyObject_CheckBuffer(o)) return false;
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_C_CONTIGUOUS | PyBUF_FORMAT) != 0) {
      PyErr_Clear();
      return false;
    }
    const char format = view.format != nullptr && view.format[0] != 0 && view.format[1] == 0
                            ? view.format[0] : 0;
    bool taken = false;
    if (format == 'i' && view.itemsize == 4)
      taken = take_values<int32_t>(view);
    else if ((format == 'l' || format == 'q') && view.itemsize == 8)
      taken = take_values<int64_t>(view);
    PyBuffer_Release(&view);
    return taken;
  }
  const T* data() const { return values_.data(); }
  int64_t size() const { return (int64_t)values_.size(); }

 private:
  static bool holds(int64_t x) { return x == (int64_t)(T)x; }

  // (a buffer need not be aligned to its type)
  template <class From>
  bool take_values(const Py_buffer& view) {
    const int64_t n = view.len / (int64_t)sizeof(From);
    const char* from = static_cast<const char*>(view.buf);
    values_.resize(n);
    if (sizeof(From) == sizeof(T)) {
      if (n > 0) std::memcpy(values_.data(), from, n * sizeof(T));
      return true;
    }
    for (int64_t i = 0; i < n; ++i) {
      From x;
      std::memcpy(&x, from + i * sizeof(From), sizeof(From));
      if (!holds(x)) return false;
      values_[i] = (T)x;
    }
    return true;
  }

  bool take_sequence(PyObject* o) {
    const Py_ssize_t n = PySequence_Fast_GET_SIZE(o);
    PyObject** items = PySequence_Fast_ITEMS(o);
    values_.resize(n);
    for (Py_ssize_t i = 0; i < n; ++i) {
      if (!PyLong_CheckExact(items[i])) return false;
      int overflow;
      const long long x = PyLong_AsLongLongAndOverflow(items[i], &overflow);
      if (overflow != 0 || !holds(x)) return false;
      values_[i] = (T)x;
    }
    return true;
  }

  c10::SmallVector<T, 72> values_;
};

// The interpreter's lock is given back in this scope, as ctypes does around a call.  (A daemon thread
// that wants it back while the interpreter is ending is ended there, by unwinding its stack: that has
// to get through the destructor, and through ordinary().)
class Unlocked {
 public:
  Unlocked() : state_(PyEval_SaveThread()) {}
  ~Unlocked() noexcept(false) { PyEval_RestoreThread(state_); }
  Unlocked(const Unlocked&) = delete;

 private:
  PyThreadState* state_;
};
static_assert(!std::is_nothrow_destructible<Unlocked>::value, "unwinding ends in an abort");

int64_t total(const HostArray<int32_t>& a) {
  int64_t sum = 0;
  for (int64_t i = 0; i < a.size(); ++i) sum += a.data()[i];
  return sum;
}

// A plain tensor (no subclass), or null.
const at::Tensor* tensor(PyObject* o) {
  return THPVariable_CheckExact(o) ? &THPVariable_Unpack(o) : nullptr;
}

bool device_array(const at::Tensor* t, at::ScalarType type, int64_t dim) {
  return t != nullptr && t->is_cuda() && t->scalar_type() == type && t->is_contiguous() &&
         (dim < 0 || t->dim() == dim);
}

bool cache(PyObject* k, PyObject* v, medha_kv_cache& kv) {
  const at::Tensor *kt = tensor(k), *vt = tensor(v);
  if (!device_array(kt, at::kBFloat16, 4) || !device_array(vt, at::kBFloat16, 4) ||
      kt->sizes() != vt->sizes())
    return false;
  for (int i = 0; i < 4; ++i)
    if (kt->size(i) > std::numeric_limits<int32_t>::max()) return false;
  kv = medha_kv_cache{kt->data_ptr(), vt->data_ptr(), (int32_t)kt->size(0), (int32_t)kt->size(2),
                      (int32_t)kt->size(1), (int32_t)kt->size(3)};
  return true;
}

// Page table and offsets of n sequences.
bool pages(const at::Tensor* table, const HostArray<int64_t>& offs, int64_t n) {
  return device_array(table, at::kInt, -1) && n >= 1 && n < std::numeric_limits<int32_t>::max() &&
         offs.size() == n + 1 && offs.data()[n] <= table->numel();
}

// The caller's workspace, if there is one (of any type: its elements are counted as bytes).
bool room(PyObject* o, at::Tensor& t) {
  if (o == Py_None) return true;
  const at::Tensor* given = tensor(o);
  if (given == nullptr || !given->is_cuda() || !given->is_contiguous()) return false;
  t = *given;
  return true;
}

// An output: the caller's tensor, checked, or a new one.
bool output(PyObject* o, at::IntArrayRef sizes, const at::Tensor& like, at::Tensor& t) {
  if (o == Py_None) {
    t = at::empty(sizes, like.options().dtype(at::kFloat));
    return true;
  }
  const at::Tensor* given = tensor(o);
  if (!device_array(given, at::kFloat, -1) || given->sizes() != sizes) return false;
  t = *given;
  return true;
}

PyObject* pair(PyObject* a, const at::Tensor& ta, PyObject* b, const at::Tensor& tb) {
  PyObject* x = a == Py_None ? THPVariable_Wrap(ta) : Py_NewRef(a);
  PyObject* y = b == Py_None ? THPVariable_Wrap(tb) : Py_NewRef(b);
  PyObject* r = x && y ? PyTuple_Pack(2, x, y) : nullptr;
  Py_XDECREF(x);
  Py_XDECREF(y);
  return r;
}

// False without a Python error for what is no number (float() takes strings too).
bool number(PyObject* o, float& x) {
  const PyNumberMethods* as = Py_TYPE(o)->tp_as_number;
  if (as == nullptr || (as->nb_float == nullptr && as->nb_index == nullptr)) return false;
  const double d = PyFloat_AsDouble(o);
  if (d == -1.0 && PyErr_Occurred()) return false;
  x = (float)d;
  return true;
}

bool current_stream(void*& stream) {
  PyObject* s = PyObject_CallNoArgs(lib.stream);
  if (s == nullptr) return false;
  stream = PyLong_AsVoidPtr(s);
  Py_DECREF(s);
  return !PyErr_Occurred();
}

// Runs `call` as the binding's steps are run: a C++ error (a tensor without storage, memory that is
// not there) leaves the call to binding.py.  `call` returns a result, null with a Python error set,
// or null without one for "not from here".  Python errors are the caller's: the scale and the
// stream are asked for last, by Python code, where an interrupt or a signal handler's error can
// come up as well, and those do not come again on the long way.
template <class F>
PyObject* ordinary(F&& call) {
  if (lib.stream == nullptr) Py_RETURN_NONE;
  PyObject* r = nullptr;
  try {
    r = call();
  } catch (python_error& e) {
    e.restore();
  } catch (const std::exception&) {
  }
  if (r == nullptr && !PyErr_Occurred()) Py_RETURN_NONE;
  return r;
}

// Whether a library call has been made.  Its refusals come before any launch and are found again on
// the long way; other errors are raised.
bool made(int rc) {
  if (rc == MEDHA_OK) return true;
  if (rc == MEDHA_ERR_INVALID_ARG || rc == MEDHA_ERR_UNSUPPORTED || rc == MEDHA_ERR_WORKSPACE)
    return false;
  Py_XDECREF(PyObject_CallFunction(lib.check, "i", rc));
  return false;
}

at::Tensor new_workspace(size_t n, const at::TensorOptions& options) {
  return at::empty({(int64_t)std::max<size_t>(n, 256)}, options.dtype(at::kByte));
}

struct Workspace {
  at::Tensor bytes;
  at::TensorOptions options;
  std::exception_ptr error;
};

void* allocate(size_t n, void* context) {
  Workspace* w = static_cast<Workspace*>(context);
  try {
    w->bytes = new_workspace(n, w->options);
    return w->bytes.data_ptr();
  } catch (const std::exception&) {
    w->error = std::current_exception();
    return nullptr;
  }
}

// (q, k_pool, v_pool, page_table, offs, prefix_len, chunk_len, scale, out, lse, workspace)
PyObject* chunked_prefill_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return ordinary([&]() -> PyObject* {
    const at::Tensor *q, *table;
    medha_kv_cache kv;
    HostArray<int64_t> offs;
    HostArray<int32_t> pre, chk;
    float scale;
    void* stream;
    if (n != 11 || !pre.take(a[5]) || !chk.take(a[6]) || !offs.take(a[4]) ||
        !device_array(q = tensor(a[0]), at::kBFloat16, 3) || !cache(a[1], a[2], kv) ||
        q->size(2) != kv.head_dim || chk.size() != pre.size() ||
        !pages(table = tensor(a[3]), offs, pre.size()) || total(chk) != q->size(0) ||
        q->size(1) > std::numeric_limits<int32_t>::max())
      return nullptr;
    at::Tensor out, lse;
    if (!output(a[8], q->sizes(), *q, out) || !output(a[9], q->sizes().slice(0, 2), *q, lse))
      return nullptr;
    at::Tensor given;
    if (!room(a[10], given) || !number(a[7], scale) || !current_stream(stream)) return nullptr;
    Workspace ws{{}, q->options(), nullptr};
    const void* qp = q->data_ptr();
    const int32_t* tp = static_cast<const int32_t*>(table->data_ptr());
    float *op = static_cast<float*>(out.data_ptr()), *lp = static_cast<float*>(lse.data_ptr());
    void* wp = given.defined() ? given.data_ptr() : nullptr;
    const int32_t batch = (int32_t)pre.size(), h_q = (int32_t)q->size(1);
    int rc;
    {
      Unlocked unlocked;
      rc = given.defined()
               ? lib.prefill(qp, &kv, tp, offs.data(), pre.data(), chk.data(), batch, h_q, scale, op,
                             lp, wp, (size_t)given.numel(), stream)
               : lib.prefill_alloc(qp, &kv, tp, offs.data(), pre.data(), chk.data(), batch, h_q,
                                   scale, op, lp, allocate, &ws, stream);
    }
    if (ws.error) std::rethrow_exception(ws.error);
    return made(rc) ? pair(a[8], out, a[9], lse) : nullptr;
  });
}

// (q, k_pool, v_pool, page_table, offs, q_index, kv_len, scale, out, lse, workspace)
PyObject* decode_partial_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return ordinary([&]() -> PyObject* {
    const at::Tensor *q, *table;
    medha_kv_cache kv;
    HostArray<int64_t> offs;
    HostArray<int32_t> qi, kl;
    float scale;
    void* stream;
    if (n != 11 || !kl.take(a[6]) || !qi.take(a[5]) || !offs.take(a[4]) ||
        !device_array(q = tensor(a[0]), at::kBFloat16, 3) || !cache(a[1], a[2], kv) ||
        q->size(2) != kv.head_dim || kl.size() != qi.size() ||
        !pages(table = tensor(a[3]), offs, qi.size()) ||
        q->size(0) > std::numeric_limits<int32_t>::max() ||
        q->size(1) > std::numeric_limits<int32_t>::max())
      return nullptr;
    at::Tensor out, lse, ws;
    const int64_t sizes[3] = {qi.size(), q->size(1), q->size(2)};
    if (!output(a[8], at::IntArrayRef(sizes, 3), *q, out) ||
        !output(a[9], at::IntArrayRef(sizes, 2), *q, lse) || !room(a[10], ws) ||
        !number(a[7], scale) || !current_stream(stream))
      return nullptr;
    if (!ws.defined())
      ws = new_workspace(lib.decode_bytes(kl.data(), (int32_t)kl.size(), (int32_t)q->size(1),
                                          kv.num_kv_heads, kv.head_dim), q->options());
    const void* qp = q->data_ptr();
    const int32_t* tp = static_cast<const int32_t*>(table->data_ptr());
    float *op = static_cast<float*>(out.data_ptr()), *lp = static_cast<float*>(lse.data_ptr());
    void* wp = ws.data_ptr();
    int rc;
    {
      Unlocked unlocked;
      rc = lib.decode(qp, (int32_t)q->size(0), &kv, tp, offs.data(), qi.data(), kl.data(),
                    (int32_t)qi.size(), (int32_t)q->size(1), scale, op, lp, wp, (size_t)ws.numel(),
                    stream);
    }
    return made(rc) ? pair(a[8], out, a[9], lse) : nullptr;
  });
}

// (q, k_pool, v_pool, page_table, offs, q_row, chunk_len, kv_len, visible0, scale, out, lse,
// workspace)
PyObject* chunk_partial_attn(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return ordinary([&]() -> PyObject* {
    const at::Tensor *q, *table;
    medha_kv_cache kv;
    HostArray<int64_t> offs;
    HostArray<int32_t> qr, chk, kl, v0;
    float scale;
    void* stream;
    if (n != 13 || !chk.take(a[6]) || !kl.take(a[7]) || !v0.take(a[8]) ||
        !qr.take(a[5]) || !offs.take(a[4]) || !device_array(q = tensor(a[0]), at::kBFloat16, 3) ||
        !cache(a[1], a[2], kv) || q->size(2) != kv.head_dim || chk.size() != qr.size() ||
        kl.size() != qr.size() ||
        v0.size() != qr.size() || !pages(table = tensor(a[3]), offs, qr.size()) ||
        q->size(0) > std::numeric_limits<int32_t>::max() ||
        q->size(1) > std::numeric_limits<int32_t>::max())
      return nullptr;
    at::Tensor out, lse, ws;
    const int64_t sizes[3] = {total(chk), q->size(1), q->size(2)};
    if (sizes[0] < 0 || !output(a[10], at::IntArrayRef(sizes, 3), *q, out) ||
        !output(a[11], at::IntArrayRef(sizes, 2), *q, lse) || !room(a[12], ws) ||
        !number(a[9], scale) || !current_stream(stream))
      return nullptr;
    if (!ws.defined())
      ws = new_workspace(lib.chunk_bytes(chk.data(), kl.data(), (int32_t)chk.size(),
                                         (int32_t)q->size(1), kv.num_kv_heads, kv.head_dim),
                         q->options());
    const void* qp = q->data_ptr();
    const int32_t* tp = static_cast<const int32_t*>(table->data_ptr());
    float *op = static_cast<float*>(out.data_ptr()), *lp = static_cast<float*>(lse.data_ptr());
    void* wp = ws.data_ptr();
    int rc;
    {
      Unlocked unlocked;
      rc = lib.chunk(qp, (int32_t)q->size(0), &kv, tp, offs.data(), qr.data(), chk.data(), kl.data(),
                   v0.data(), (int32_t)qr.size(), (int32_t)q->size(1), scale, op, lp, wp,
                   (size_t)ws.numel(), stream);
    }
    return made(rc) ? pair(a[10], out, a[11], lse) : nullptr;
  });
}

// (out_partial, lse_partial, out, lse)
PyObject* lse_merge(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return ordinary([&]() -> PyObject* {
    const at::Tensor *po, *pl;
    void* stream;
    if (n != 4 || !device_array(po = tensor(a[0]), at::kFloat, 4) ||
        !device_array(pl = tensor(a[1]), at::kFloat, 3) || pl->sizes() != po->sizes().slice(0, 3) ||
        po->size(0) > std::numeric_limits<int32_t>::max() ||
        po->size(2) > std::numeric_limits<int32_t>::max() ||
        po->size(3) > std::numeric_limits<int32_t>::max())
      return nullptr;
    at::Tensor out, lse;
    if (!output(a[2], po->sizes().slice(1), *po, out) ||
        !output(a[3], po->sizes().slice(1, 2), *po, lse) || !current_stream(stream))
      return nullptr;
    const float *pop = static_cast<const float*>(po->data_ptr()),
                *plp = static_cast<const float*>(pl->data_ptr());
    float *op = static_cast<float*>(out.data_ptr()), *lp = static_cast<float*>(lse.data_ptr());
    int rc;
    {
      Unlocked unlocked;
      rc = lib.merge(pop, plp, (int32_t)po->size(0), po->size(1), (int32_t)po->size(2),
                   (int32_t)po->size(3), op, lp, stream);
    }
    return made(rc) ? pair(a[2], out, a[3], lse) : nullptr;
  });
}

// (k_new, v_new, k_pool, v_pool, page_table, offs, prefix_len, chunk_len); True when done
PyObject* kv_append(PyObject*, PyObject* const* a, Py_ssize_t n) {
  return ordinary([&]() -> PyObject* {
    const at::Tensor *k, *v, *table;
    medha_kv_cache kv;
    HostArray<int64_t> offs;
    HostArray<int32_t> pre, chk;
    void* stream;
    if (n != 8 || !pre.take(a[6]) || !chk.take(a[7]) || !offs.take(a[5]) ||
        !device_array(k = tensor(a[0]), at::kBFloat16, 3) ||
        !device_array(v = tensor(a[1]), at::kBFloat16, 3) || k->sizes() != v->sizes() ||
        !cache(a[2], a[3], kv) || k->size(1) != kv.num_kv_heads || k->size(2) != kv.head_dim ||
        chk.size() != pre.size() ||
        !pages(table = tensor(a[4]), offs, pre.size()) || total(chk) != k->size(0) ||
        !current_stream(stream))
      return nullptr;
    const void *kp = k->data_ptr(), *vp = v->data_ptr();
    const int32_t* tp = static_cast<const int32_t*>(table->data_ptr());
    int rc;
    {
      Unlocked unlocked;
      rc = lib.append(kp, vp, &kv, tp, offs.data(), pre.data(), chk.data(), (int32_t)pre.size(),
                    stream);
    }
    return made(rc) ? Py_NewRef(Py_True) : nullptr;
  });
}

// bind(stream, check, entry points' addresses in the order below)
PyObject* bind(PyObject*, PyObject* const* a, Py_ssize_t n) {
  constexpr int kEntries = 8;
  if (n != 2 + kEntries) {
    PyErr_Format(PyExc_TypeError, "bind() takes %d arguments", 2 + kEntries);
    return nullptr;
  }
  void* p[kEntries];
  for (int i = 0; i < kEntries; ++i) p[i] = PyLong_AsVoidPtr(a[i + 2]);
  if (PyErr_Occurred()) return nullptr;
  lib.prefill = reinterpret_cast<decltype(lib.prefill)>(p[0]);
  lib.prefill_alloc = reinterpret_cast<decltype(lib.prefill_alloc)>(p[1]);
  lib.decode = reinterpret_cast<decltype(lib.decode)>(p[2]);
  lib.decode_bytes = reinterpret_cast<decltype(lib.decode_bytes)>(p[3]);
  lib.chunk = reinterpret_cast<decltype(lib.chunk)>(p[4]);
  lib.chunk_bytes = reinterpret_cast<decltype(lib.chunk_bytes)>(p[5]);
  lib.merge = reinterpret_cast<decltype(lib.merge)>(p[6]);
  lib.append = reinterpret_cast<decltype(lib.append)>(p[7]);
  Py_XSETREF(lib.stream, Py_NewRef(a[0]));
  Py_XSETREF(lib.check, Py_NewRef(a[1]));
  Py_RETURN_NONE;
}

#define CALL(name) {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(name)), METH_FASTCALL, nullptr}
PyMethodDef methods[] = {CALL(bind), CALL(chunked_prefill_attn), CALL(decode_partial_attn),
                         CALL(chunk_partial_attn), CALL(lse_merge), CALL(kv_append),
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  PyObject* m = PyModule_Create(&module);
  if (m && PyModule_AddStringConstant(m, "torch_version", MEDHA_TORCH_VERSION) != 0) Py_CLEAR(m);
  return m;
}
