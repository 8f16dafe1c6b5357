// bind.cpp -- the execute calls of the Python binding (ar.py) in native code.
//
// A call passes up to 128 rank tensors.  Checking each of them and reading
// its address in Python cost 0.14 us per rank and 4 us per call, most of the
// time of a small Allreduce; here it is 0.02 us per rank.  The checks are
// those of ar._ptr_table, made anew on every call (nothing is kept from one
// call to the next).  Whatever fails one, or is no plain torch tensor in a
// list or tuple -- raw addresses, subclasses, other sequences -- is answered
// with None, and the caller takes the Python path, which names the fault.
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

#include "../../include/ar.h"

namespace {

using ExecuteFn = ar_status (*)(ar_plan*, void* const*, int64_t, int64_t, hipStream_t);
ExecuteFn g_execute[2] = {nullptr, nullptr};  // ar_execute_batched, ar_execute_noalloc; set once, at import

constexpr Py_ssize_t kMaxRanks = 128;
constexpr int64_t kMaxExtent = int64_t(1) << 46;

// Reads an int argument; false (no error set) if it is none or does not fit.
bool as_int(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  int overflow = 0;
  const long long x = PyLong_AsLongLongAndOverflow(o, &overflow);
  if (overflow != 0 || (x == -1 && PyErr_Occurred())) {
    PyErr_Clear();
    return false;
  }
  *v = x;
  return true;
}

// Whether tensor t can serve as a rank buffer of `extent` elements of the
// plan's dtype (0 int32, 1 float32, < 0 any of 4 bytes) on GPU `device`.
bool rank_buffer(const at::Tensor& t, int64_t extent, int64_t dtype, int64_t device) {
  if (extent == 0) return true;
  if (!t.is_cuda() || t.get_device() != device) return false;
  const auto st = t.scalar_type();
  if (dtype == 0 ? st != at::kInt : dtype == 1 ? st != at::kFloat : t.element_size() != 4) return false;
  if (t.layout() != at::kStrided || !t.is_contiguous() || !t.has_storage()) return false;
  const int64_t have = int64_t(t.storage().nbytes() / 4) - t.storage_offset();
  return have >= extent;
}

// execute(handle, (P, n, dtype), buffers, batch, stride, device, stream, which)
// -> status, or None where the Python path has to look.
PyObject* execute(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  if (nargs != 8 || !PyTuple_CheckExact(args[1]) || PyTuple_GET_SIZE(args[1]) != 3) Py_RETURN_NONE;
  int64_t handle, P, n, dtype = -1, batch, stride, device, stream, which;
  PyObject* dt = PyTuple_GET_ITEM(args[1], 2);
  if (!as_int(args[0], &handle) || !as_int(PyTuple_GET_ITEM(args[1], 0), &P) ||
      !as_int(PyTuple_GET_ITEM(args[1], 1), &n) || (dt != Py_None && !as_int(dt, &dtype)) ||
      !as_int(args[3], &batch) || !as_int(args[4], &stride) || !as_int(args[5], &device) ||
      !as_int(args[6], &stream) || !as_int(args[7], &which) || which < 0 || which > 1 || g_execute[which] == nullptr)
    Py_RETURN_NONE;
  PyObject* seq = args[2];
  const bool list = PyList_CheckExact(seq);
  if (!list && !PyTuple_CheckExact(seq)) Py_RETURN_NONE;
  if (P < 1 || P > kMaxRanks || Py_SIZE(seq) != P || n < 0 || batch < 1 || stride < 0) Py_RETURN_NONE;
  const int64_t step = batch == 1 && stride < n ? n : stride;
  if (n > kMaxExtent || (step > 0 && batch - 1 > (kMaxExtent - n) / step)) Py_RETURN_NONE;
  const int64_t extent = n > 0 ? (batch - 1) * step + n : 0;
  void* table[kMaxRanks];
  try {
    for (Py_ssize_t x = 0; x < P; ++x) {
      PyObject* o = list ? PyList_GET_ITEM(seq, x) : PyTuple_GET_ITEM(seq, x);
      if (!THPVariable_CheckExact(o)) Py_RETURN_NONE;
      const at::Tensor& t = THPVariable_Unpack(o);
      if (!rank_buffer(t, extent, dtype, device)) Py_RETURN_NONE;
      table[x] = t.data_ptr();
    }
  } catch (...) {  // a tensor without an address of its own: the Python path raises
    Py_RETURN_NONE;
  }
  ar_status st;
  Py_BEGIN_ALLOW_THREADS
  st = g_execute[which](reinterpret_cast<ar_plan*>(handle), table, batch, stride, reinterpret_cast<hipStream_t>(stream));
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(long(st));
}

// bind(address of ar_execute_batched, address of ar_execute_noalloc): the
// functions of the library that ar.py loaded.
PyObject* bind(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  int64_t a, b;
  if (nargs != 2 || !as_int(args[0], &a) || !as_int(args[1], &b)) {
    PyErr_SetString(PyExc_TypeError, "bind takes two addresses");
    return nullptr;
  }
  g_execute[0] = reinterpret_cast<ExecuteFn>(a);
  g_execute[1] = reinterpret_cast<ExecuteFn>(b);
  Py_RETURN_NONE;
}

PyMethodDef kMethods[] = {
    {"execute", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(execute)), METH_FASTCALL, nullptr},
    {"bind", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(bind)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_arbind", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__arbind(void) { return PyModule_Create(&kModule); }
