// How a C function of a Python module runs C++ code (call_path.cpp).
#pragma once

#define PY_SSIZE_T_CLEAN
#include <Python.h>

#include <cxxabi.h>

#include <exception>

namespace heatkv {

// A thread that is in a call when the interpreter ends is unwound and gone as soon as it takes the interpreter's lock: not
// out of a destructor, which would end the process, nor into a handler that keeps what it catches, which would do the same.

// f() with the interpreter's lock released.
template <class F>
int without_lock(const F& f) {
  int rc = 0;
  std::exception_ptr error;
  PyThreadState* const state = PyEval_SaveThread();
  try {
    rc = f();
  } catch (const abi::__forced_unwind&) {
    throw;
  } catch (...) {
    error = std::current_exception();
  }
  PyEval_RestoreThread(state);
  if (error) std::rethrow_exception(error);
  return rc;
}

// F(a, n), or None where it throws: a C++ exception must not reach the interpreter's C frames.
template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyObject* guarded(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    return F(a, n);
  } catch (const abi::__forced_unwind&) {
    throw;
  } catch (...) {
  }
  PyErr_Clear();  // after the exception is gone: one that came from Python holds its error until then
  Py_RETURN_NONE;
}

template <PyObject* (*F)(PyObject* const*, Py_ssize_t)>
PyCFunction fastcall() {
  return reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(guarded<F>));
}

}  // namespace heatkv
