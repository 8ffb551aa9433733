// Module call_lock: C functions made as those of _heatkv_call, without a library behind them.
#include "python_calls.h"

#include <unistd.h>

#include <stdexcept>

namespace {

PyObject* wait(PyObject* const* a, Py_ssize_t n) {
  const long us = n == 1 ? PyLong_AsLong(a[0]) : 0;
  return PyLong_FromLong(heatkv::without_lock([&] { return usleep(us); }));
}

PyObject* fail(PyObject* const*, Py_ssize_t) {
  return PyLong_FromLong(heatkv::without_lock([]() -> int { throw std::runtime_error("without the lock"); }));
}

PyMethodDef methods[] = {{"wait", heatkv::fastcall<wait>(), METH_FASTCALL, nullptr},
                         {"fail", heatkv::fastcall<fail>(), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "call_lock", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_call_lock() { return PyModule_Create(&module); }
