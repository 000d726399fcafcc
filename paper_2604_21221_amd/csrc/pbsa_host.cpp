// Calls a libpbsa function with Python arguments: the marshalling of the binding (pbsa.py), in native code.  A call
// takes up to two dozen tensors and a step makes four calls, which is what a small step costs on the host: 0.25 us per
// tensor and 3 us for the stream in Python, against about 0.02 us per argument here.
#include <ATen/TensorSubclassLikeUtils.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

constexpr int kMaxArgs = 26;   // of pbsa_attention_fwd_plan_split, the longest

PyObject* g_params = nullptr;       // the types of pbsa_params and pbsa_grid, set once
PyObject* g_grid = nullptr;
PyObject* g_array = nullptr;        // ctypes.Array

enum class Take { yes, no, error };  // no: not one of the plain cases, error: a Python error is set

// The address of the bytes of a ctypes object; the caller holds it for the length of the call.
Take bytes_of(PyObject* o, int64_t& out) {
  Py_buffer view;
  if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return Take::error;
  out = reinterpret_cast<int64_t>(view.buf);
  PyBuffer_Release(&view);
  return Take::yes;
}

// The value of an argument of the given kind (pbsa.py's _SIGNATURES), in the plain cases.
Take convert(char kind, PyObject* o, int64_t& out) {
  switch (kind) {
    case 'p': return Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(g_params) ? bytes_of(o, out) : Take::no;
    case 'g': return Py_TYPE(o) == reinterpret_cast<PyTypeObject*>(g_grid) ? bytes_of(o, out) : Take::no;
    case 'P':
    case 'L': {
      const int is = PyObject_IsInstance(o, g_array);
      return is < 0 ? Take::error : is ? bytes_of(o, out) : Take::no;
    }
    case 'i':
    case 'l':
    case 'z':
      if (!PyLong_CheckExact(o)) return Take::no;
      break;
    case 't':
      if (THPVariable_CheckExact(o)) {
        const at::Tensor& t = THPVariable_Unpack(o);
        if (!t.is_cuda() || (t.dim() < 3 && !t.is_contiguous())) return Take::no;
        out = reinterpret_cast<int64_t>(t.data_ptr());
        return Take::yes;
      }
      [[fallthrough]];
    case 'w':
      if (o == Py_None) {
        out = 0;
        return Take::yes;
      }
      if (!PyLong_Check(o)) return Take::no;
      break;
    default: return Take::no;
  }
  out = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(o));
  return PyErr_Occurred() ? Take::error : Take::yes;
}

// invoke(function address, kinds, *arguments) -> the function's int result, or NotImplemented with nothing called where
// an argument is not one of the plain cases of its kind.  Every argument of the library's functions is an integer or a
// pointer; the calling convention of this platform lets a function be called with more of those than it looks at
// (registers first, the caller cleans the stack), so one call expression serves all of them.
PyObject* invoke(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS                         // a tensor without memory of its own (of a function transform, say) throws
  if (n < 2 || n - 2 > kMaxArgs || !PyLong_CheckExact(args[0]) || !PyBytes_CheckExact(args[1]) || PyBytes_GET_SIZE(args[1]) != n - 2) {
    PyErr_SetString(PyExc_TypeError, "pbsa: wrong number of arguments");
    return nullptr;
  }
  const char* const kinds = PyBytes_AS_STRING(args[1]);
  int64_t f, a[kMaxArgs] = {};
  f = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(args[0]));
  for (Py_ssize_t i = 0; i < n - 2; ++i) {
    const Take t = convert(kinds[i], args[i + 2], a[i]);
    if (t == Take::error) return nullptr;
    if (t == Take::no) Py_RETURN_NOTIMPLEMENTED;
  }
  typedef int (*fn_t)(int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                      int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                      int64_t, int64_t, int64_t, int64_t);
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<fn_t>(f)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13],
                                    a[14], a[15], a[16], a[17], a[18], a[19], a[20], a[21], a[22], a[23], a[24], a[25]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

// plain_rows(Kl, Vl, H, Nq, d, watched, *tensors) -> bool: whether each of the tensors (None is passed over) can be read as it
// is: exactly a torch.Tensor, bf16 on Kl's device, strided, [H][Nq][d] with rows that are contiguous, aligned to 16 bytes and
// no overlap of each other, without a pending negation or, where autograd watches, a gradient to follow, and not in Kl's or
// Vl's own memory.  (The same questions asked from Python took 3 us of a small step's 28 on the host.)
PyObject* plain_rows(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS
  if (n < 6 || !THPVariable_Check(args[0]) || !THPVariable_Check(args[1]) || !PyBool_Check(args[5])) {
    PyErr_SetString(PyExc_TypeError, "pbsa: plain_rows takes two tensors, three sizes, a flag and tensors");
    return nullptr;
  }
  const at::Tensor& kl = THPVariable_Unpack(args[0]);
  const at::Tensor& vl = THPVariable_Unpack(args[1]);
  int64_t size[3];
  for (int i = 0; i < 3; ++i) {
    size[i] = PyLong_AsLongLong(args[2 + i]);
    if (size[i] == -1 && PyErr_Occurred()) return nullptr;
  }
  const bool watched = args[5] == Py_True;
  for (Py_ssize_t i = 6; i < n; ++i) {
    if (args[i] == Py_None) continue;
    if (Py_TYPE(args[i]) != reinterpret_cast<PyTypeObject*>(THPVariableClass)) Py_RETURN_FALSE;
    const at::Tensor& x = THPVariable_Unpack(args[i]);
    if (at::isTensorSubclassLike(x) || x.scalar_type() != at::kBFloat16 || x.layout() != at::kStrided || x.device() != kl.device() ||
        x.dim() != 3 || (watched && x.requires_grad()) || x.is_neg() || !x.has_storage())
      Py_RETURN_FALSE;
    for (int k = 0; k < 3; ++k)
      if (x.size(k) != size[k]) Py_RETURN_FALSE;
    const void* const mem = x.storage().unsafeGetStorageImpl();
    if (mem == kl.storage().unsafeGetStorageImpl() || mem == vl.storage().unsafeGetStorageImpl()) Py_RETURN_FALSE;
    if (x.stride(2) != 1 || x.stride(0) % 8 || x.stride(1) % 8 || x.stride(1) < size[2] || reinterpret_cast<uintptr_t>(x.data_ptr()) % 16)
      Py_RETURN_FALSE;
  }
  Py_RETURN_TRUE;
  END_HANDLE_TH_ERRORS
}

// setup(type of pbsa_params, type of pbsa_grid, ctypes.Array)
PyObject* setup(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 3 || !PyType_Check(args[0]) || !PyType_Check(args[1]) || !PyType_Check(args[2])) {
    PyErr_SetString(PyExc_TypeError, "pbsa: setup takes three types");
    return nullptr;
  }
  PyObject** const to[3] = {&g_params, &g_grid, &g_array};
  for (int i = 0; i < 3; ++i) {
    Py_INCREF(args[i]);
    Py_XDECREF(*to[i]);
    *to[i] = args[i];
  }
  Py_RETURN_NONE;
}

template <typename F>
constexpr PyCFunction fast(F f) {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(f));
}
PyMethodDef methods[] = {
    {"invoke", fast(invoke), METH_FASTCALL, "invoke(function address, kinds, *arguments) -> int or NotImplemented"},
    {"plain_rows", fast(plain_rows), METH_FASTCALL, "plain_rows(Kl, Vl, H, Nq, d, watched, *tensors) -> bool"},
    {"setup", fast(setup), METH_FASTCALL, "setup(pbsa_params, pbsa_grid, ctypes.Array)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pbsa_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pbsa_host() { return PyModule_Create(&module); }
