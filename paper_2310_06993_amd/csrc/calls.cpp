// Native argument marshalling for binding.py: the functions there whose work is done by a kernel or two take longer to
// marshal through ctypes than to launch (MI355X host, per call: torch.cuda.current_stream() 2.8 us, five tensor
// arguments 0.9 us, the ctypes call itself 1.0 us; a launch 2.9 us).  Every function here has the name, the arguments
// and the defaults of its C entry point's Python form, takes torch tensors (or None) for device pointers and raises
// what binding.check raises.  No arithmetic and no state beyond the addresses handed over by bind().
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>
#include <string>
#include <utility>

#include "../../include/optireduce.h"

namespace {

PyObject* g_check = nullptr;     // check(status, name): raises for a status other than OR_OK
PyObject* g_array = nullptr;     // ctypes.Array
PyObject* g_address = nullptr;   // address(obj) -> int or None, for descriptors that are no ctypes array
PyObject* g_integer = nullptr;   // integer(obj, unsigned) -> int, for what is neither an int nor has __index__
PyObject* g_extent = nullptr;    // extent(obj) -> (address, bytes), for what is no torch tensor but behaves like one
PyObject* g_cuda_stream = nullptr;

constexpr int kMaxArgs = 12;

template <class A>
A as(uint64_t v) {
  if constexpr (std::is_pointer_v<A>) return reinterpret_cast<A>(static_cast<uintptr_t>(v));
  else return static_cast<A>(v);
}
template <class... A, size_t... I>
or_status invoke(or_status (*f)(A...), const uint64_t* v, std::index_sequence<I...>) {
  return f(as<A>(v[I])...);
}
template <class... A>
or_status invoke(or_status (*f)(A...), const uint64_t* v) {
  return invoke(f, v, std::index_sequence_for<A...>{});
}

// One entry point.  `kinds`, one letter per Python argument: t tensor or None -> pointer, w the same -> pointer and
// byte size, b host array of descriptors, i/u integer, q truth value, s stream.  The arguments from `required` on are
// optional (None).
struct Entry {
  const char* name;
  const char* kinds;
  int required;
  const char* args[kMaxArgs];
  or_status (*call)(void*, const uint64_t*);
  void* fn;
};
#define OR_ENTRY(NAME, KINDS, REQUIRED, ...)                                                                     \
  {#NAME, KINDS, REQUIRED, {__VA_ARGS__}, [](void* f, const uint64_t* v) { return invoke((decltype(&NAME))f, v); }, nullptr}
#define OR_PATH(NAME, FIRST)                                                                                        \
  OR_ENTRY(NAME, "ttiuiuuttws", 8, FIRST, "masks", "N", "shard_len", "block_log2", "seed", "base_index", "out", "count_out", \
           "workspace", "stream")

Entry g_entries[] = {
    OR_ENTRY(or_rht_encode, "tuiuts", 5, "grad", "n", "block_log2", "seed", "out", "stream"),
    OR_ENTRY(or_rht_encode_at, "tuiuuts", 6, "grad", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_rht_encode_bf16, "tuiuuts", 6, "grad", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_masked_reduce, "ttiutts", 6, "shards", "masks", "N", "shard_len", "sum_out", "count_out", "stream"),
    OR_ENTRY(or_masked_reduce_bf16, "ttiutts", 6, "shards", "masks", "N", "shard_len", "sum_out", "count_out", "stream"),
    OR_ENTRY(or_rht_decode, "tuiuts", 5, "agg", "n", "block_log2", "seed", "out", "stream"),
    OR_ENTRY(or_rht_decode_at, "tuiuuts", 6, "agg", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_rht_decode_bf16, "tuiuuts", 6, "agg", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_finalize_decode, "ttuiuuts", 7, "total", "count", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_finalize_decode_bf16, "ttuiuuts", 7, "total", "count", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_PATH(or_reduce_decode, "shards"),
    OR_PATH(or_reduce_decode_bf16, "shards"),
    OR_PATH(or_fused_path, "grads"),
    OR_PATH(or_fused_path_bf16, "grads"),
    OR_ENTRY(or_fused_path_bf16_static, "ttiuiuutts", 8, "grads", "masks", "N", "shard_len", "block_log2", "seed", "base_index",
             "out", "count_out", "stream"),
    OR_ENTRY(or_fused_path_batched, "biiiqws", 5, "buckets", "n_buckets", "N", "block_log2", "bf16", "workspace", "stream"),
    OR_ENTRY(or_fused_path_batched_monitored, "biiiqtws", 6, "buckets", "n_buckets", "N", "block_log2", "bf16", "totals",
             "workspace", "stream"),
    OR_ENTRY(or_reduce_decode_batched, "biiiqtws", 5, "buckets", "n_buckets", "N", "block_log2", "bf16", "totals", "workspace",
             "stream"),
    OR_ENTRY(or_masked_reduce_batched, "biiqs", 4, "buckets", "n_buckets", "N", "bf16", "stream"),
    OR_ENTRY(or_finalize_decode_batched, "biiqs", 4, "buckets", "n_buckets", "block_log2", "bf16", "stream"),
    OR_ENTRY(or_finalize, "ttuts", 4, "total", "count", "shard_len", "mean_out", "stream"),
    OR_ENTRY(or_finalize_bf16, "ttuts", 4, "total", "count", "shard_len", "mean_out", "stream"),
    OR_ENTRY(or_received_total, "tuts", 3, "count", "shard_len", "total_out", "stream"),
    OR_ENTRY(or_rht_decode_masked, "ttuiuuts", 7, "agg", "mask", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_rht_decode_masked_bf16, "ttuiuuts", 7, "agg", "mask", "n", "block_log2", "seed", "base_index", "out", "stream"),
    OR_ENTRY(or_masked_reduce_pairs, "tttiutts", 7, "sums", "counts", "masks", "G", "shard_len", "sum_out", "count_out", "stream"),
};
constexpr int kEntries = sizeof(g_entries) / sizeof(g_entries[0]);

// an int-like object that has no need of ctypes' rules
bool index_of(PyObject* o, uint64_t& v) {
  if (PyLong_Check(o)) {
    v = PyLong_AsUnsignedLongLongMask(o);
  } else {
    PyObject* i = PyNumber_Index(o);
    if (!i) return false;
    v = PyLong_AsUnsignedLongLongMask(i);
    Py_DECREF(i);
  }
  return !(v == (uint64_t)-1 && PyErr_Occurred());
}

// an int-like result of a helper (None counts as 0); steals the reference
bool take_int(PyObject* o, uint64_t& v) {
  if (!o) return false;
  bool ok = true;
  if (o == Py_None) v = 0;
  else ok = index_of(o, v);
  Py_DECREF(o);
  return ok;
}

bool int_arg(PyObject* o, bool is_unsigned, uint64_t& v) {
  if (PyIndex_Check(o)) return index_of(o, v);
  return take_int(PyObject_CallFunctionObjArgs(g_integer, o, is_unsigned ? Py_True : Py_False, nullptr), v);
}

bool tensor_arg(PyObject* o, uint64_t& ptr, uint64_t* bytes) {
  ptr = 0;
  if (bytes) *bytes = 0;
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) {
    PyObject* pair = PyObject_CallFunctionObjArgs(g_extent, o, bytes ? Py_True : Py_False, nullptr);
    if (!pair) return false;
    unsigned long long p = 0, n = 0;
    const bool ok = PyArg_ParseTuple(pair, "KK", &p, &n);
    Py_DECREF(pair);
    ptr = p;
    if (bytes) *bytes = n;
    return ok;
  }
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda()) {
    PyErr_SetString(PyExc_ValueError, "liboptireduce_hip takes device tensors");
    return false;
  }
  if (!t.is_contiguous()) {
    PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
    return false;
  }
  ptr = (uint64_t)(uintptr_t)t.mutable_data_ptr();   // as Tensor.data_ptr(): a copy-on-write clone gets storage of its own
  if (bytes) *bytes = (uint64_t)t.numel() * t.element_size();
  return true;
}

bool stream_arg(PyObject* o, uint64_t& v) {
  if (o == Py_None) {
    v = (uint64_t)(uintptr_t)c10::hip::getCurrentHIPStream().stream();
    return true;
  }
  if (PyObject* s = PyObject_GetAttr(o, g_cuda_stream)) return take_int(s, v);
  if (!PyErr_ExceptionMatches(PyExc_AttributeError)) return false;
  PyErr_Clear();
  return take_int(PyNumber_Long(o), v);
}

// held or given up for a scope, whichever way it is left
struct Buffer {
  Py_buffer view = {};
  ~Buffer() {
    if (view.obj) PyBuffer_Release(&view);
  }
};
struct WithoutGil {
  PyThreadState* state = PyEval_SaveThread();
  ~WithoutGil() { PyEval_RestoreThread(state); }
};

PyObject* run(const Entry& e, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  const int n = (int)strlen(e.kinds);
  PyObject* got[kMaxArgs] = {};
  if (nargs > n) return PyErr_Format(PyExc_TypeError, "%s() takes at most %d arguments (%zd given)", e.name, n, nargs);
  for (Py_ssize_t i = 0; i < nargs; ++i) got[i] = args[i];
  for (Py_ssize_t k = 0, nk = kwnames ? PyTuple_GET_SIZE(kwnames) : 0; k < nk; ++k) {
    PyObject* name = PyTuple_GET_ITEM(kwnames, k);
    int i = 0;
    while (i < n && PyUnicode_CompareWithASCIIString(name, e.args[i]) != 0) ++i;
    if (i == n) return PyErr_Format(PyExc_TypeError, "%s() got an unexpected keyword argument '%U'", e.name, name);
    if (got[i]) return PyErr_Format(PyExc_TypeError, "%s() got multiple values for argument '%s'", e.name, e.args[i]);
    got[i] = args[nargs + k];
  }
  uint64_t v[kMaxArgs + 1];
  int nv = 0;
  Buffer buffer;
  bool ok = true;
  for (int i = 0; ok && i < n; ++i) {
    PyObject* o = got[i];
    if (!o) {
      if (i < e.required) {
        PyErr_Format(PyExc_TypeError, "%s() missing required argument: '%s'", e.name, e.args[i]);
        ok = false;
        break;
      }
      o = Py_None;
    }
    switch (e.kinds[i]) {
      case 't': ok = tensor_arg(o, v[nv], nullptr); ++nv; break;
      case 'w': ok = tensor_arg(o, v[nv], &v[nv + 1]); nv += 2; break;
      case 'i':
      case 'u': ok = int_arg(o, e.kinds[i] == 'u', v[nv]); ++nv; break;
      case 'q': {
        const int t = PyObject_IsTrue(o);
        ok = t >= 0;
        v[nv++] = t > 0;
        break;
      }
      case 's': ok = stream_arg(o, v[nv]); ++nv; break;
      case 'b':
        // (a ctypes pointer offers a buffer too, but that is the pointer itself)
        if (PyObject_TypeCheck(o, (PyTypeObject*)g_array)) {
          ok = PyObject_GetBuffer(o, &buffer.view, PyBUF_SIMPLE) == 0;
          v[nv++] = ok ? (uint64_t)(uintptr_t)buffer.view.buf : 0;
        } else {
          ok = take_int(PyObject_CallFunctionObjArgs(g_address, o, nullptr), v[nv]);
          ++nv;
        }
        break;
    }
  }
  if (!ok) return nullptr;
  or_status s;
  {
    WithoutGil released;
    s = e.call(e.fn, v);
  }
  if (s == OR_OK) Py_RETURN_NONE;
  return PyObject_CallFunction(g_check, "is", (int)s, e.name);
}

template <int I>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs, PyObject* kwnames) {
  try {
    if (g_entries[I].fn) return run(g_entries[I], args, nargs, kwnames);
    PyErr_SetString(PyExc_RuntimeError, "bind() has not been called");
  } catch (const std::exception& e) {   // torch reports errors of the HIP runtime this way
    PyErr_SetString(PyExc_RuntimeError, e.what());
  }
  return nullptr;
}

// bind(addresses: dict name -> int, check, ctypes.Array, address, integer, extent)
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *addresses, *check, *array, *address, *integer, *extent;
  if (!PyArg_ParseTuple(args, "O!OO!OOO", &PyDict_Type, &addresses, &check, &PyType_Type, &array, &address, &integer, &extent))
    return nullptr;
  for (Entry& e : g_entries) {
    PyObject* a = PyDict_GetItemString(addresses, e.name);
    if (!a) return PyErr_Format(PyExc_KeyError, "%s", e.name);
    uint64_t v;
    if (!index_of(a, v)) return nullptr;
    e.fn = (void*)(uintptr_t)v;
  }
  for (auto [global, value] : {std::pair{&g_check, check}, {&g_array, array}, {&g_address, address}, {&g_integer, integer}, {&g_extent, extent}}) {
    Py_INCREF(value);
    Py_XSETREF(*global, value);
  }
  Py_RETURN_NONE;
}

PyMethodDef g_methods[kEntries + 2];
std::string g_docs[kEntries];   // the signature, in the form that inspect reads

std::string signature(const Entry& e) {
  std::string s = std::string(e.name) + "($module";
  for (int i = 0; e.kinds[i]; ++i) s += std::string(", ") + e.args[i] + (i >= e.required ? "=None" : "");
  return s + ")\n--\n\n";
}

template <size_t... I>
void fill_methods(std::index_sequence<I...>) {
  ((g_docs[I] = signature(g_entries[I])), ...);
  ((g_methods[I] = {g_entries[I].name, (PyCFunction)(void (*)(void))entry<(int)I>, METH_FASTCALL | METH_KEYWORDS, g_docs[I].c_str()}), ...);
  g_methods[kEntries] = {"bind", bind, METH_VARARGS, nullptr};
  g_methods[kEntries + 1] = {nullptr, nullptr, 0, nullptr};
}

PyModuleDef g_module = {PyModuleDef_HEAD_INIT, "_calls", nullptr, -1, g_methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__calls() {
  fill_methods(std::make_index_sequence<kEntries>{});
  g_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  return g_cuda_stream ? PyModule_Create(&g_module) : nullptr;
}
