// Argument marshalling of the per-step calls (binding.py): one Python call checks the tensors, takes
// their addresses and calls the library's C entry point, without the interpreter in between.
//
// What bounds a small step that is called eagerly is the host: a launch costs about 2.5 us, and ctypes with
// the checks written in Python added 1.2 to 2.2 us to each call.  Measured (a step of four calls, 128 fp32
// tokens, top-2, host time without waiting; layout / dispatch / expert stand-in / combine): 3.8 / 4.1 / 4.5 /
// 4.7 us that way, 3.4 / 3.6 / 3.9 / 4.1 this way, the step 17.9 and 16.3.
#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <stdint.h>

namespace {

PyObject *name_contiguous, *name_data_ptr, *name_cuda_stream;

// Device address of a tensor (must be contiguous), an int, or None.
bool pointer_of(PyObject* o, uint64_t* out) {
  if (o == Py_None) {
    *out = 0;
    return true;
  }
  if (!PyLong_Check(o)) {
    PyObject* whole = PyObject_CallMethodNoArgs(o, name_contiguous);
    if (whole == nullptr) return false;
    const int yes = PyObject_IsTrue(whole);
    Py_DECREF(whole);
    if (yes < 0) return false;
    if (yes == 0) {
      PyErr_SetString(PyExc_ValueError, "tensor must be contiguous");
      return false;
    }
    PyObject* address = PyObject_CallMethodNoArgs(o, name_data_ptr);
    if (address == nullptr) return false;
    *out = PyLong_AsUnsignedLongLongMask(address);
    Py_DECREF(address);
  } else {
    *out = PyLong_AsUnsignedLongLongMask(o);
  }
  return !(*out == (uint64_t)-1 && PyErr_Occurred());
}

// A stream's raw handle, or None for the default stream.
bool stream_of(PyObject* o, uint64_t* out) {
  if (o == Py_None || PyLong_Check(o)) return pointer_of(o, out);
  PyObject* handle = PyObject_GetAttr(o, name_cuda_stream);
  if (handle == nullptr) return false;
  *out = PyLong_AsUnsignedLongLongMask(handle);
  Py_DECREF(handle);
  return !(*out == (uint64_t)-1 && PyErr_Occurred());
}

// call(entry point's address, "kinds of its arguments", arguments...) -> its return code.  Kinds: p a device
// address (tensor, int or None), i an int32, h a handle as an int, s the stream.  Every argument is of the
// integer class, so it travels in a 64-bit register or stack slot whatever its width.
constexpr int kMost = 9;
PyObject* call(PyObject*, PyObject* const* args, Py_ssize_t nargs) {
  Py_ssize_t n = 0;
  const char* kinds = nargs >= 2 ? PyUnicode_AsUTF8AndSize(args[1], &n) : nullptr;
  if (kinds == nullptr || n != nargs - 2 || n < 1 || n > kMost) {
    if (!PyErr_Occurred()) PyErr_SetString(PyExc_TypeError, "call(address, kinds, arguments...)");
    return nullptr;
  }
  const uint64_t entry = PyLong_AsUnsignedLongLong(args[0]);
  if (entry == (uint64_t)-1 && PyErr_Occurred()) return nullptr;
  uint64_t a[kMost] = {};
  for (Py_ssize_t i = 0; i < n; ++i) {
    PyObject* o = args[i + 2];
    bool ok = true;
    switch (kinds[i]) {
      case 'p': ok = pointer_of(o, &a[i]); break;
      case 's': ok = stream_of(o, &a[i]); break;
      default: {
        PyObject* number = PyNumber_Index(o);
        if (number == nullptr) return nullptr;
        a[i] = PyLong_AsUnsignedLongLongMask(number);
        Py_DECREF(number);
        ok = !(a[i] == (uint64_t)-1 && PyErr_Occurred());
      }
    }
    if (!ok) return nullptr;
  }
  int code;
  typedef int (*Entry)(uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t, uint64_t,
                       uint64_t);
  Py_BEGIN_ALLOW_THREADS  // (arguments past the entry point's own are not looked at)
  code = reinterpret_cast<Entry>(entry)(a[0], a[1], a[2], a[3], a[4], a[5], a[6], a[7], a[8]);
  Py_END_ALLOW_THREADS
  return PyLong_FromLong(code);
}

PyMethodDef methods[] = {{"call", (PyCFunction)(void (*)(void))call, METH_FASTCALL,
                          "call(address, kinds, arguments...) -> return code"},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_marshal", nullptr, -1, methods,
                      nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__marshal() {
  name_contiguous = PyUnicode_InternFromString("is_contiguous");
  name_data_ptr = PyUnicode_InternFromString("data_ptr");
  name_cuda_stream = PyUnicode_InternFromString("cuda_stream");
  if (!name_contiguous || !name_data_ptr || !name_cuda_stream) return nullptr;
  return PyModule_Create(&module);
}
