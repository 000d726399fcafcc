// Calls a libpbsa function with Python arguments: the marshalling of the binding (pbsa.py), in native code.  A call
// takes up to two dozen tensors and a step makes four calls, which is what a small step costs on the host: 0.25 us per
// tensor and 3 us for the stream in Python, against about 0.02 us per argument here.
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>

namespace {

constexpr int kMaxArgs = 26;   // of pbsa_attention_fwd_plan, the longest, 25

PyObject* g_host_types = nullptr;   // (ctypes.Structure, ctypes.Array): what is passed by the address of its bytes

// The value a C argument gets: a device address for a tensor, the address of its bytes for a ctypes structure or
// array, an integer for itself, 0 for None.  False: a Python error is set.
bool convert(PyObject* o, int64_t& out) {
  if (o == Py_None) {
    out = 0;
  } else if (THPVariable_Check(o)) {
    const at::Tensor& t = THPVariable_Unpack(o);
    if (!t.is_cuda()) {
      PyErr_SetString(PyExc_TypeError, "pbsa: tensor arguments must live on the GPU");
      return false;
    }
    if (t.dim() < 3 && !t.is_contiguous()) {
      PyErr_SetString(PyExc_TypeError, "pbsa: small tensors must be contiguous");
      return false;
    }
    out = reinterpret_cast<int64_t>(t.data_ptr());
  } else if (PyLong_Check(o)) {
    out = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(o));
    if (PyErr_Occurred()) return false;
  } else if (PyObject_IsInstance(o, g_host_types) == 1) {
    Py_buffer view;
    if (PyObject_GetBuffer(o, &view, PyBUF_SIMPLE) != 0) return false;
    out = reinterpret_cast<int64_t>(view.buf);   // the caller holds the object for the length of the call
    PyBuffer_Release(&view);
  } else {                                       // an integer of another kind; anything else is refused here
    PyObject* i = PyNumber_Index(o);
    if (!i) return false;
    out = static_cast<int64_t>(PyLong_AsUnsignedLongLongMask(i));
    Py_DECREF(i);
    if (PyErr_Occurred()) return false;
  }
  return true;
}

// invoke(function address, *arguments) -> the function's int result.  Every argument of the library's functions is an
// integer or a pointer; the calling convention of this platform lets a function be called with more of those than it
// looks at (registers first, the caller cleans the stack), so one call expression serves all of them.
PyObject* invoke(PyObject*, PyObject* const* args, Py_ssize_t n) {
  HANDLE_TH_ERRORS                         // a tensor without memory of its own (of a function transform, say) throws
  if (n < 1 || n - 1 > kMaxArgs) {
    PyErr_SetString(PyExc_TypeError, "pbsa: wrong number of arguments");
    return nullptr;
  }
  int64_t v[kMaxArgs + 1] = {};
  for (Py_ssize_t i = 0; i < n; ++i)
    if (!convert(args[i], v[i])) return nullptr;
  typedef int (*fn_t)(int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                      int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t, int64_t,
                      int64_t, int64_t, int64_t, int64_t);
  const int64_t* a = v + 1;
  int rc;
  Py_BEGIN_ALLOW_THREADS
  rc = reinterpret_cast<fn_t>(v[0])(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8], a[9], a[10], a[11], a[12], a[13],
                                    a[14], a[15], a[16], a[17], a[18], a[19], a[20], a[21], a[22], a[23], a[24], a[25]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(rc);
  END_HANDLE_TH_ERRORS
}

PyMethodDef methods[] = {
    {"invoke", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(invoke)), METH_FASTCALL,
     "invoke(function address, *arguments) -> int"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_pbsa_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__pbsa_host() {
  PyObject* ct = PyImport_ImportModule("ctypes");
  if (!ct) return nullptr;
  PyObject* s = PyObject_GetAttrString(ct, "Structure");
  PyObject* a = PyObject_GetAttrString(ct, "Array");
  Py_DECREF(ct);
  if (!s || !a) return nullptr;
  g_host_types = PyTuple_Pack(2, s, a);
  Py_DECREF(s);
  Py_DECREF(a);
  return g_host_types ? PyModule_Create(&module) : nullptr;
}
