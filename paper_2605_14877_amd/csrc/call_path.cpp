// Python module _heatkv_call: the per-layer calls of binding.py without the interpreter in between.
//
// A generation pass makes one or two library calls per layer and scale, and below about 300 tokens the kernels are
// shorter than the 10 us that operand checks, stream lookup and argument conversion took in Python and ctypes (2.1, 2.9
// and 2.0 us, next to 3.7 us for the library call itself, 3.2 of them the launch).  The functions here do the same
// checks on the tensors and call the library.  They return its error code, or None for anything that is not plainly
// in order: the caller then takes the Python path, which names the mistake.  A tensor may answer a question about itself with
// an exception (one without sizes, a subclass with a sizes policy of its own): that is not plainly in order either.
#include "python_calls.h"

#include <ATen/hip/impl/HIPStreamMasqueradingAsCUDA.h>
#include <torch/csrc/autograd/python_variable.h>

#include <cstdint>
#include <new>
#include <vector>

#include "heatkv.h"

namespace {

constexpr const char* kPlanName = "heatkv_plan_info";

// What the operands of a plan's calls must look like.
struct PlanInfo {
  heatkv_plan* plan;
  int64_t L, H, d, batch, dtype;
  std::vector<int64_t> t;
  int64_t arena_bytes;
};

void free_plan_info(PyObject* capsule) {
  delete static_cast<PlanInfo*>(PyCapsule_GetPointer(capsule, kPlanName));
}

// plan_info(handle, L, H, d, batch, dtype, t, arena_bytes) -> capsule
PyObject* plan_info(PyObject*, PyObject* args) try {
  unsigned long long handle;
  long long L, H, d, batch, dtype, arena_bytes;
  PyObject* t;
  if (!PyArg_ParseTuple(args, "KLLLLLO!L", &handle, &L, &H, &d, &batch, &dtype, &PyTuple_Type, &t, &arena_bytes))
    return nullptr;
  std::vector<int64_t> tokens;
  for (Py_ssize_t i = 0; i < PyTuple_GET_SIZE(t); ++i) {
    const long long n = PyLong_AsLongLong(PyTuple_GET_ITEM(t, i));
    if (n == -1 && PyErr_Occurred()) return nullptr;
    tokens.push_back(n);
  }
  auto* info = new PlanInfo{reinterpret_cast<heatkv_plan*>(handle), L, H, d, batch, dtype, std::move(tokens), arena_bytes};
  PyObject* capsule = PyCapsule_New(info, kPlanName, free_plan_info);
  if (!capsule) delete info;
  return capsule;
} catch (const std::bad_alloc&) {
  return PyErr_NoMemory();
}

// Address and size of a contiguous device tensor; None is a null pointer.
bool device_tensor(PyObject* o, const at::Tensor** tensor, void** ptr) {
  *tensor = nullptr;
  *ptr = nullptr;
  if (o == Py_None) return true;
  if (!THPVariable_Check(o)) return false;
  const at::Tensor& x = THPVariable_Unpack(o);
  if (!x.is_cuda() || !x.is_contiguous()) return false;
  *tensor = &x;
  *ptr = x.data_ptr();
  return true;
}

bool operand(PyObject* o, at::IntArrayRef shape, int64_t dtype, void** ptr) {
  const at::Tensor* x;
  if (!device_tensor(o, &x, ptr)) return false;
  return !x || (x->scalar_type() == (dtype == HEATKV_BF16 ? at::kBFloat16 : at::kFloat) && x->sizes() == shape);
}

bool buffer(PyObject* o, int64_t min_bytes, void** ptr, size_t* bytes) {
  const at::Tensor* x;
  if (!device_tensor(o, &x, ptr)) return false;
  const int64_t n = x ? x->numel() * static_cast<int64_t>(x->element_size()) : 0;
  if (bytes) *bytes = static_cast<size_t>(n);
  return !x || n >= min_bytes;
}

bool integer(PyObject* o, long* v) {
  *v = PyLong_AsLong(o);
  return !(*v == -1 && PyErr_Occurred());
}

bool number(PyObject* o, float* v) {
  *v = static_cast<float>(PyFloat_AsDouble(o));
  return !PyErr_Occurred();
}

bool stream_of(PyObject* o, void** stream) {
  if (o == Py_None) {
    *stream = c10::hip::getCurrentHIPStreamMasqueradingAsCUDA().stream();
    return true;
  }
  if (!PyLong_Check(o)) return false;
  *stream = PyLong_AsVoidPtr(o);
  return !PyErr_Occurred();
}

PyObject* not_plain() {
  PyErr_Clear();
  Py_RETURN_NONE;
}

// scale_call(plan_info, which, layer, k, q, k_cur, v_cur, k_arena, v_arena, sm_scale, out, ws, stream)
// which: 0 append_scale (q, sm_scale, out and ws unused), 1 attend_scale, 2 attend_append_scale
PyObject* scale_call(PyObject* const* a, Py_ssize_t n) {
  if (n != 13) return not_plain();
  auto* info = static_cast<PlanInfo*>(PyCapsule_GetPointer(a[0], kPlanName));
  long which, layer, k;
  if (!info || !integer(a[1], &which) || !integer(a[2], &layer) || !integer(a[3], &k)) return not_plain();
  if (layer < 0 || layer >= info->L || k < 0 || k >= static_cast<long>(info->t.size())) return not_plain();
  const int64_t shape[4] = {info->batch, info->H, info->t[k], info->d};
  void *q = nullptr, *kc, *vc, *ka, *va, *out = nullptr, *ws = nullptr, *stream;
  size_t ws_bytes = 0;
  float sm = 0.f;
  if (!operand(a[5], shape, info->dtype, &kc) || !operand(a[6], shape, info->dtype, &vc) ||
      !buffer(a[7], info->arena_bytes, &ka, nullptr) || !buffer(a[8], info->arena_bytes, &va, nullptr) ||
      !stream_of(a[12], &stream))
    return not_plain();
  if (which != 0 && (!operand(a[4], shape, info->dtype, &q) || !number(a[9], &sm) ||
                     !operand(a[10], shape, info->dtype, &out) || !buffer(a[11], 0, &ws, &ws_bytes)))
    return not_plain();
  return PyLong_FromLong(heatkv::without_lock([&] {
    if (which == 0) return heatkv_append_scale(info->plan, layer, k, kc, vc, ka, va, stream);
    if (which == 1) return heatkv_attend_scale(info->plan, layer, k, q, kc, vc, ka, va, sm, out, ws, ws_bytes, stream);
    return heatkv_attend_append_scale(info->plan, layer, k, q, kc, vc, ka, va, sm, out, ws, ws_bytes, stream);
  }));
}

const heatkv_shape* shape_at(PyObject* o) {
  const auto* s = static_cast<const heatkv_shape*>(PyLong_AsVoidPtr(o));
  return s && s->t && s->K >= 1 && s->K <= HEATKV_MAX_SCALES ? s : nullptr;
}

bool calibrate_operands(const heatkv_shape* s, long k1, PyObject* q, PyObject* k_all, PyObject* mass, void** qp, void** kp,
                        void** mp) {
  if (k1 < 0 || k1 >= s->K) return false;
  int64_t c = 0;
  for (long k = 0; k <= k1; ++k) c += s->t[k];
  const int64_t q_shape[4] = {s->batch, s->H, s->t[k1], s->d}, k_shape[4] = {s->batch, s->H, c, s->d};
  const int64_t m_shape[3] = {s->batch, s->H, s->K};
  return operand(q, q_shape, s->dtype, qp) && operand(k_all, k_shape, s->dtype, kp) &&
         operand(mass, m_shape, HEATKV_F32, mp);
}

bool beta_operand(const heatkv_shape* s, PyObject* beta, void** ptr) {
  const int64_t shape[4] = {s->L, s->H, s->K, s->K};
  return operand(beta, shape, HEATKV_F32, ptr);
}

// calibrate_call(address of the heatkv_shape, which, layer, k1, q, k_all, sm_scale, weight, beta, mass, ws, stream)
// which: 0 calibrate, 1 calibrate_static (ws unused), 2 calibrate_accumulate
PyObject* calibrate_call(PyObject* const* a, Py_ssize_t n) {
  if (n != 12) return not_plain();
  const heatkv_shape* s = shape_at(a[0]);
  long which, layer, k1;
  float sm, weight;
  void *q, *k_all, *beta, *mass, *ws, *stream;
  size_t ws_bytes;
  if (!s || !integer(a[1], &which) || !integer(a[2], &layer) || !integer(a[3], &k1) || !number(a[6], &sm) ||
      !number(a[7], &weight) || !calibrate_operands(s, k1, a[4], a[5], a[9], &q, &k_all, &mass) ||
      !beta_operand(s, a[8], &beta) || !buffer(a[10], 0, &ws, &ws_bytes) || !stream_of(a[11], &stream))
    return not_plain();
  return PyLong_FromLong(heatkv::without_lock([&] {
    float* const m = static_cast<float*>(mass);
    if (which == 0) return heatkv_calibrate(s, layer, k1, q, k_all, sm, m, ws, ws_bytes, stream);
    if (which == 1) return heatkv_calibrate_static(s, layer, k1, q, k_all, sm, m, stream);
    return heatkv_calibrate_accumulate(s, layer, k1, q, k_all, sm, weight, static_cast<float*>(beta), m, ws, ws_bytes,
                                       stream);
  }));
}

// calibrate_scales_call(address of the heatkv_shape, layer, k1 list, q list, k_all list, sm_scale, weight, beta,
//                       mass list or None, ws, stream); the lists have one length
PyObject* calibrate_scales_call(PyObject* const* a, Py_ssize_t n) {
  if (n != 11) return not_plain();
  const heatkv_shape* s = shape_at(a[0]);
  long layer;
  float sm, weight;
  void *beta, *ws, *stream;
  size_t ws_bytes;
  if (!s || !integer(a[1], &layer) || !PyList_Check(a[2]) || !PyList_Check(a[3]) || !PyList_Check(a[4]) ||
      !(a[8] == Py_None || PyList_Check(a[8])) || !number(a[5], &sm) || !number(a[6], &weight) ||
      !beta_operand(s, a[7], &beta) || !buffer(a[9], 0, &ws, &ws_bytes) || !stream_of(a[10], &stream))
    return not_plain();
  const Py_ssize_t scales = PyList_GET_SIZE(a[2]);
  if (scales < 1 || scales > s->K || PyList_GET_SIZE(a[3]) != scales || PyList_GET_SIZE(a[4]) != scales ||
      (a[8] != Py_None && PyList_GET_SIZE(a[8]) != scales))
    return not_plain();
  int32_t k1[HEATKV_MAX_SCALES];
  void *q[HEATKV_MAX_SCALES], *k_all[HEATKV_MAX_SCALES], *mass[HEATKV_MAX_SCALES];
  for (Py_ssize_t i = 0; i < scales; ++i) {
    long k;
    PyObject* m = a[8] == Py_None ? Py_None : PyList_GET_ITEM(a[8], i);
    if (!integer(PyList_GET_ITEM(a[2], i), &k) ||
        !calibrate_operands(s, k, PyList_GET_ITEM(a[3], i), PyList_GET_ITEM(a[4], i), m, &q[i], &k_all[i], &mass[i]))
      return not_plain();
    k1[i] = static_cast<int32_t>(k);
  }
  return PyLong_FromLong(heatkv::without_lock([&] {
    return heatkv_calibrate_scales_accumulate(s, layer, static_cast<int>(scales), k1, q, k_all, sm, weight,
                                              static_cast<float*>(beta),
                                              a[8] == Py_None ? nullptr : reinterpret_cast<float* const*>(mass), ws, ws_bytes,
                                              stream);
  }));
}

PyMethodDef methods[] = {{"plan_info", plan_info, METH_VARARGS, nullptr},
                         {"scale_call", heatkv::fastcall<scale_call>(), METH_FASTCALL, nullptr},
                         {"calibrate_call", heatkv::fastcall<calibrate_call>(), METH_FASTCALL, nullptr},
                         {"calibrate_scales_call", heatkv::fastcall<calibrate_scales_call>(), METH_FASTCALL, nullptr},
                         {nullptr, nullptr, 0, nullptr}};

PyModuleDef module = {PyModuleDef_HEAD_INIT, "_heatkv_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__heatkv_call() { return PyModule_Create(&module); }
