// Native half of the Python binding (diffopt.py, tree.py): argument checks,
// address extraction and the C ABI call of one entry point in one function
// call, and the host part of a tree operation over a list of leaves.
//
// In Python an entry point spent about 0.6 us on the checks of each operand
// and 3 us in ctypes (the 5-step leaf-direct driver on a 6-leaf tree: 12 us a
// call, its kernel 3.7 us); leaf_pointers replaces a Python loop, a tensor
// built from a list of ints and a copy into pinned memory.
//
// Every function here handles the ordinary case (plain tensors and parameters
// that pass every check) and returns None for anything else; the Python
// caller then takes its own path, which accepts or refuses the arguments with
// its own messages.  No check is remembered from one call to the next.
#include <torch/csrc/autograd/python_variable.h>
#include <torch/torch.h>

#include <algorithm>
#include <cstdint>
#include <type_traits>
#include <utility>
#include <vector>

#include "diffopt.h"

namespace {

// An argument that the ordinary path does not take.
struct Other {};

// The tensor an object is, if it is exactly a torch.Tensor or a Parameter.
const at::Tensor& tensor_of(PyObject* o) {
  if (!THPVariable_CheckExact(o)) throw Other{};
  return THPVariable_Unpack(o);
}

constexpr int64_t kAnyCount = -1;  // an operand of any number of elements

// Address of a contiguous device tensor of this type with n elements; None is
// the null pointer, an int an address.
void* address(PyObject* o, at::ScalarType type, int64_t n) {
  if (o == Py_None) return nullptr;
  if (PyLong_CheckExact(o)) {
    void* p = PyLong_AsVoidPtr(o);
    if (!p && PyErr_Occurred()) {
      PyErr_Clear();
      throw Other{};
    }
    return p;
  }
  const at::Tensor& t = tensor_of(o);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous() || (n != kAnyCount && t.numel() != n)) throw Other{};
  return t.data_ptr();
}

constexpr Py_ssize_t kMaxList = 256;  // entries of one operand list on the ordinary path

// One C argument made from one Python argument.
struct Slot {
  void* p = nullptr;
  int64_t i = 0;
  double d = 0.0;
  void* list[kMaxList];
};

template <class T>
struct Arg;

template <class T, at::ScalarType TYPE>
struct PointerArg {
  static T get(Slot& s) { return static_cast<T>(s.p); }
  static void set(Slot& s, PyObject* o, int64_t n) { s.p = address(o, TYPE, n); }
};
template <>
struct Arg<const float*> : PointerArg<const float*, at::kFloat> {};
template <>
struct Arg<float*> : PointerArg<float*, at::kFloat> {};
template <>
struct Arg<const uint64_t*> : PointerArg<const uint64_t*, at::kLong> {};

// A host array of addresses, from a list or tuple.
template <class T, at::ScalarType TYPE>
struct ListArg {
  static T get(Slot& s) { return reinterpret_cast<T>(s.list); }
  static void set(Slot& s, PyObject* o, int64_t n) {
    if (!PyList_CheckExact(o) && !PyTuple_CheckExact(o)) throw Other{};
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(o);
    if (k > kMaxList) throw Other{};
    PyObject** items = PySequence_Fast_ITEMS(o);
    for (Py_ssize_t j = 0; j < k; ++j) s.list[j] = address(items[j], TYPE, n);
  }
};
template <>
struct Arg<const float* const*> : ListArg<const float* const*, at::kFloat> {};
template <>
struct Arg<float* const*> : ListArg<float* const*, at::kFloat> {};
template <>
struct Arg<const uint64_t* const*> : ListArg<const uint64_t* const*, at::kLong> {};

// Opaque addresses: a segment table's handle, a stream.
template <class T>
struct HandleArg {
  static T get(Slot& s) { return static_cast<T>(s.p); }
  static void set(Slot& s, PyObject* o, int64_t) {
    if (o != Py_None && !PyLong_CheckExact(o)) throw Other{};
    s.p = address(o, at::kLong, kAnyCount);
  }
};
template <>
struct Arg<const diffopt_segtable*> : HandleArg<const diffopt_segtable*> {};
template <>
struct Arg<void*> : HandleArg<void*> {};

template <class T>
struct IntArg {
  static T get(Slot& s) { return static_cast<T>(s.i); }
  static void set(Slot& s, PyObject* o, int64_t) {
    if (!PyLong_Check(o)) throw Other{};
    s.i = std::is_unsigned_v<T> ? static_cast<int64_t>(PyLong_AsUnsignedLongLong(o)) : PyLong_AsLongLong(o);
    if ((s.i == -1 && PyErr_Occurred()) || (sizeof(T) == 4 && s.i != static_cast<int32_t>(s.i))) {
      PyErr_Clear();
      throw Other{};
    }
  }
};
template <>
struct Arg<int64_t> : IntArg<int64_t> {};
template <>
struct Arg<uint64_t> : IntArg<uint64_t> {};
template <>
struct Arg<int32_t> : IntArg<int32_t> {};

template <>
struct Arg<double> {
  static double get(Slot& s) { return s.d; }
  static void set(Slot& s, PyObject* o, int64_t) {
    if (PyFloat_CheckExact(o)) {
      s.d = PyFloat_AS_DOUBLE(o);
    } else if (PyLong_Check(o)) {
      s.d = PyLong_AsDouble(o);
      if (s.d == -1.0 && PyErr_Occurred()) {
        PyErr_Clear();
        throw Other{};
      }
    } else {
      throw Other{};
    }
  }
};

template <class... A, size_t... I>
int invoke(int (*fn)(A...), Slot* s, PyObject* const* args, int64_t n, std::index_sequence<I...>) {
  (Arg<A>::set(s[I], args[I], n), ...);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = fn(Arg<A>::get(s[I])...);
  Py_END_ALLOW_THREADS
  return rc;
}

template <class... A>
PyObject* call(int (*fn)(A...), PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != static_cast<Py_ssize_t>(sizeof...(A)) + 1) {
    PyErr_SetString(PyExc_TypeError, "wrong number of arguments");
    return nullptr;
  }
  try {
    Slot count;
    if (args[0] != Py_None) Arg<int64_t>::set(count, args[0], 0);
    if (count.i < 0) throw Other{};  // no tensor has that many elements
    const int64_t n = args[0] == Py_None ? kAnyCount : count.i;
    Slot slots[sizeof...(A)];
    return PyLong_FromLong(invoke(fn, slots, args + 1, n, std::index_sequence_for<A...>{}));
  } catch (...) {  // an argument of another kind, or a tensor without storage
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// (n, then the C arguments) -> return code, or None: n is the element count
// that every tensor operand must have (None: any).
template <auto FN>
PyObject* entry(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  return call(FN, args, nargs);
}

// The interpreter lock given up for a scope.
struct Unlocked {
  PyThreadState* state = PyEval_SaveThread();
  ~Unlocked() { PyEval_RestoreThread(state); }
};

// leaf_pointers(groups, device index) -> list with, per group of leaves, a
// device int64 tensor of their addresses (None for None): slices of one device
// tensor, filled by one asynchronous copy from pinned host memory on the
// current stream.  The addresses are listed under the interpreter lock, the
// allocations and the copy, which can wait for the runtime, run without it.
PyObject* leaf_pointers(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 2 || (!PyList_CheckExact(args[0]) && !PyTuple_CheckExact(args[0]))) Py_RETURN_NONE;
  PyObject* out = nullptr;
  try {
    const long device = PyLong_AsLong(args[1]);
    if (device == -1 && PyErr_Occurred()) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    const Py_ssize_t k = PySequence_Fast_GET_SIZE(args[0]);
    PyObject** groups = PySequence_Fast_ITEMS(args[0]);
    std::vector<int64_t> addresses, lengths(static_cast<size_t>(k), -1);  // -1: None
    for (Py_ssize_t g = 0; g < k; ++g) {
      if (groups[g] == Py_None) continue;
      if (!PyList_CheckExact(groups[g]) && !PyTuple_CheckExact(groups[g])) throw Other{};
      const Py_ssize_t len = PySequence_Fast_GET_SIZE(groups[g]);
      PyObject** leaves = PySequence_Fast_ITEMS(groups[g]);
      for (Py_ssize_t j = 0; j < len; ++j) {
        const at::Tensor& t = tensor_of(leaves[j]);
        if (!t.is_contiguous()) throw Other{};
        addresses.push_back(reinterpret_cast<int64_t>(t.data_ptr()));
      }
      lengths[static_cast<size_t>(g)] = len;
    }
    at::Tensor dev;
    {
      const Unlocked unlocked;
      const auto opts = at::TensorOptions().dtype(at::kLong);
      const at::Tensor host = at::empty({static_cast<int64_t>(addresses.size())}, opts.pinned_memory(true));
      std::copy(addresses.begin(), addresses.end(), host.data_ptr<int64_t>());
      dev = host.to(opts.device(at::kCUDA, static_cast<at::DeviceIndex>(device)), /*non_blocking=*/true);
    }
    out = PyList_New(k);
    if (!out) return nullptr;
    int64_t at = 0;
    for (Py_ssize_t g = 0; g < k; ++g) {
      const int64_t len = lengths[static_cast<size_t>(g)];
      if (len < 0) {
        Py_INCREF(Py_None);
        PyList_SET_ITEM(out, g, Py_None);
        continue;
      }
      PyObject* t = THPVariable_Wrap(dev.narrow(0, at, len));
      if (!t) {
        Py_DECREF(out);
        return nullptr;
      }
      PyList_SET_ITEM(out, g, t);
      at += len;
    }
    return out;
  } catch (...) {
    Py_XDECREF(out);
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// leaf_shapes(leaves) -> tuple of the leaves' shapes (tuples of ints) if they
// are plain tensors of one dtype on one device, else None.
PyObject* leaf_shapes(PyObject*, PyObject* leaves) {
  if (!PyList_CheckExact(leaves) || PyList_GET_SIZE(leaves) == 0) Py_RETURN_NONE;
  const Py_ssize_t k = PyList_GET_SIZE(leaves);
  PyObject* out = PyTuple_New(k);
  if (!out) return nullptr;
  try {
    const at::Tensor& first = tensor_of(PyList_GET_ITEM(leaves, 0));
    for (Py_ssize_t j = 0; j < k; ++j) {
      const at::Tensor& t = tensor_of(PyList_GET_ITEM(leaves, j));
      if (t.scalar_type() != first.scalar_type() || t.device() != first.device()) throw Other{};
      const auto sizes = t.sizes();
      PyObject* shape = PyTuple_New(static_cast<Py_ssize_t>(sizes.size()));
      if (!shape) {
        Py_DECREF(out);
        return nullptr;
      }
      PyTuple_SET_ITEM(out, j, shape);
      for (size_t d = 0; d < sizes.size(); ++d) {
        PyObject* v = PyLong_FromLongLong(sizes[d]);
        if (!v) {
          Py_DECREF(out);
          return nullptr;
        }
        PyTuple_SET_ITEM(shape, static_cast<Py_ssize_t>(d), v);
      }
    }
    return out;
  } catch (...) {
    Py_DECREF(out);
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

#define ENTRY(name) \
  {#name, reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&entry<&diffopt_##name>)), METH_FASTCALL, nullptr}

PyMethodDef methods[] = {
    ENTRY(adam_fwd),
    ENTRY(adam_bwd),
    ENTRY(adam_unrolled_fwd),
    ENTRY(adam_unrolled_bwd),
    ENTRY(adam_fwd_tree),
    ENTRY(adam_bwd_tree),
    ENTRY(adam_unrolled_fwd_tree),
    ENTRY(adam_unrolled_bwd_tree),
    ENTRY(sgd_fwd),
    ENTRY(sgd_bwd),
    ENTRY(rmsprop_fwd),
    ENTRY(rmsprop_bwd),
    ENTRY(sgd_fwd_tree),
    ENTRY(sgd_bwd_tree),
    ENTRY(rmsprop_fwd_tree),
    ENTRY(rmsprop_bwd_tree),
    ENTRY(es_perturb),
    ENTRY(es_estimate),
    ENTRY(es_perturb_gaussian),
    ENTRY(es_estimate_gaussian),
    ENTRY(es_weights),
    {"leaf_pointers", reinterpret_cast<PyCFunction>(reinterpret_cast<void*>(&leaf_pointers)), METH_FASTCALL, nullptr},
    {"leaf_shapes", &leaf_shapes, METH_O, nullptr},
    {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_binding", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__binding(void) { return PyModule_Create(&module); }
