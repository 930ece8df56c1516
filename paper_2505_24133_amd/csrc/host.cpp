// Host side of an appended token in native code.  A decode loop calls this once per token, and the kernel behind it runs 2 us, so
// what the call costs on the host is what the loop waits for: with the checks, the parameter block and the call through ctypes in
// Python 7.5 us an append (one sequence of 32 layers, DecodeCache.append), now 3.7, 2.6 of them the launch; 128 appends and the
// compression behind them 1200 us, now 710, and over tokens and a cache that were never used before 1370, now 850.
// Directly behind a burst of other launches and a synchronization (a thousand small kernels are enough) both take longer, 1540 and
// 1270: for the next millisecond a thread of the runtime retires what was launched before, and a launch of any kind costs twice as
// much beside it.
//
// append() takes a call whose arguments are all in order and enqueues it; anything else (another type, a subclass of the shape or of a
// tensor, another layout or device, a paged cache, a value out of an int's range) it does not touch
// and answers None, and the Python binding goes through its own checks.
#include <Python.h>

#include <ATen/core/Tensor.h>
#include <c10/hip/HIPFunctions.h>
#include <c10/hip/HIPStream.h>
#include <torch/csrc/autograd/python_variable.h>

#include "rkv.h"

namespace {

using AppendFn = rkv_status (*)(const rkv_params*, void*, void*, void*, const void*, const void*, const void*, int32_t, int32_t, void*);
AppendFn append_fn = nullptr;
PyObject* shape_type = nullptr;    // rkv.Shape

enum Field { kProblems, kKvHeads, kQHeads, kTokens, kBudget, kAlpha, kHeadDim, kPoolW, kBeta, kThreshold, kLam, kEps, kFlags, kPageSize, kFields };
const char* const kNames[kFields] = {"num_problems", "kv_heads", "q_heads", "n_tokens", "budget", "alpha", "head_dim",
                                     "pool_w", "beta", "sim_threshold", "lam", "eps", "flags", "page_size"};
PyObject* names[kFields];

// One field of the shape as it lies in the parameter block: an int inside its range, or a float.
bool int_field(PyObject* shape, Field f, int64_t lo, int64_t hi, int64_t* out) {
  PyObject* v = PyObject_GetAttr(shape, names[f]);
  if (v == nullptr) return false;
  const bool is_int = PyLong_CheckExact(v);
  int over = 0;
  *out = is_int ? PyLong_AsLongLongAndOverflow(v, &over) : 0;
  Py_DECREF(v);
  return is_int && over == 0 && *out >= lo && *out <= hi;
}
bool float_field(PyObject* shape, Field f, float* out) {
  PyObject* v = PyObject_GetAttr(shape, names[f]);
  if (v == nullptr) return false;
  const bool is_float = PyFloat_CheckExact(v);
  *out = is_float ? (float)PyFloat_AS_DOUBLE(v) : 0.f;
  Py_DECREF(v);
  return is_float;
}

// A plain strided bf16 tensor in GPU memory with the given sizes; `dense`: contiguous, else only its last dimension.
const at::Tensor* plain(PyObject* o, at::IntArrayRef sizes, bool dense) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.is_cuda() || t.layout() != at::kStrided || !t.has_storage() || t.scalar_type() != at::kBFloat16 ||
      t.sizes() != sizes || (dense ? !t.is_contiguous() : t.stride(3) != 1))
    return nullptr;
  return &t;
}

PyObject* append(PyObject*, PyObject* const* args, Py_ssize_t count) {
  if (count != 9) {
    PyErr_SetString(PyExc_TypeError, "append takes a shape, six tensors, a position and a slot");
    return nullptr;
  }
  try {
    PyObject* shape = args[0];
    constexpr int64_t kMax = INT32_MAX;
    int64_t n[kFields] = {};
    rkv_params p = {};
    // (a subclass may fill the parameter block in its own way)
    bool ok = append_fn != nullptr && (PyObject*)Py_TYPE(shape) == shape_type;
    for (Field f : {kProblems, kKvHeads, kQHeads, kTokens, kBudget, kAlpha, kHeadDim, kPoolW, kBeta}) ok = ok && int_field(shape, f, -kMax - 1, kMax, &n[f]);
    ok = ok && int_field(shape, kFlags, 0, UINT32_MAX, &n[kFlags]) && int_field(shape, kPageSize, 0, 0, &n[kPageSize]);
    ok = ok && float_field(shape, kThreshold, &p.sim_threshold) && float_field(shape, kLam, &p.lambda) && float_field(shape, kEps, &p.eps);
    int over_at = 0, over_slot = 0;
    ok = ok && PyLong_CheckExact(args[7]) && PyLong_CheckExact(args[8]);
    const long long at_row = ok ? PyLong_AsLongLongAndOverflow(args[7], &over_at) : 0, slot = ok ? PyLong_AsLongLongAndOverflow(args[8], &over_slot) : 0;
    ok = ok && over_at == 0 && over_slot == 0 && at_row >= -kMax && at_row <= kMax && slot >= -kMax && slot <= kMax;
    if (PyErr_Occurred()) PyErr_Clear();                 // (a shape without one of the fields: the binding answers that)
    if (!ok) Py_RETURN_NONE;
    const int64_t P = n[kProblems], H = n[kKvHeads], Hq = n[kQHeads], N = n[kTokens], d = n[kHeadDim];
    const at::Tensor* k = plain(args[1], {P, H, N, d}, false);
    const at::Tensor* v = plain(args[2], {P, H, N, d}, false);
    const at::Tensor* q = plain(args[3], {P, Hq, n[kAlpha], d}, false);
    const at::Tensor* k_new = plain(args[4], {P, H, d}, true);
    const at::Tensor* v_new = plain(args[5], {P, H, d}, true);
    const at::Tensor* q_new = plain(args[6], {P, Hq, d}, true);
    if (!k || !v || !q || !k_new || !v_new || !q_new) Py_RETURN_NONE;
    const int device = c10::hip::current_device();       // whose stream is used
    for (const at::Tensor* t : {k, v, q, k_new, v_new, q_new})
      if (t->get_device() != device) Py_RETURN_NONE;
    p.num_problems = (int32_t)P; p.kv_heads = (int32_t)H; p.q_heads = (int32_t)Hq; p.n_tokens = (int32_t)N; p.head_dim = (int32_t)d;
    p.alpha = (int32_t)n[kAlpha]; p.budget = (int32_t)n[kBudget]; p.pool_w = (int32_t)n[kPoolW]; p.beta = (int32_t)n[kBeta];
    p.flags = (uint32_t)n[kFlags];
    p.k_stride_problem = k->stride(0); p.k_stride_head = k->stride(1); p.k_stride_token = k->stride(2);
    p.v_stride_problem = v->stride(0); p.v_stride_head = v->stride(1); p.v_stride_token = v->stride(2);
    if (!q->is_contiguous()) { p.q_stride_problem = q->stride(0); p.q_stride_head = q->stride(1); p.q_stride_token = q->stride(2); }
    void *kp = k->data_ptr(), *vp = v->data_ptr(), *qp = q->data_ptr(), *kn = k_new->data_ptr(), *vn = v_new->data_ptr(), *qn = q_new->data_ptr();
    void* stream = c10::hip::getCurrentHIPStream().stream();
    rkv_status s;
    // (a launch can wait for room in its queue; the caller holds references to all arguments)
    Py_BEGIN_ALLOW_THREADS
    s = append_fn(&p, kp, vp, qp, kn, vn, qn, (int32_t)at_row, (int32_t)slot, stream);
    Py_END_ALLOW_THREADS
    return PyLong_FromLong(s);
  } catch (const std::exception& e) {
    PyErr_SetString(PyExc_RuntimeError, e.what());
    return nullptr;
  }
}

// The address of rkv_cache_append in the loaded library and the class of its shapes.
PyObject* bind(PyObject*, PyObject* args) {
  PyObject *address, *type;
  if (!PyArg_ParseTuple(args, "OO!", &address, &PyType_Type, &type)) return nullptr;
  void* p = PyLong_AsVoidPtr(address);
  if (p == nullptr && PyErr_Occurred()) return nullptr;
  append_fn = reinterpret_cast<AppendFn>(p);
  Py_INCREF(type);
  Py_XDECREF(shape_type);
  shape_type = type;
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {
    {"append", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(append)), METH_FASTCALL,
     "append(shape, k_cache, v_cache, q_cache, k_new, v_new, q_new, position, slot) -> status, or None if the call is not taken"},
    {"bind", bind, METH_VARARGS, "bind(address of rkv_cache_append, class of the shapes)"},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__host() {
  for (int f = 0; f < kFields; ++f)
    if ((names[f] = PyUnicode_InternFromString(kNames[f])) == nullptr) return nullptr;
  return PyModule_Create(&module);
}
