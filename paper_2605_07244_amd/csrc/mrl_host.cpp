// Host side of the calls that take a few microseconds on the GPU, as a CPython extension: checks the tensors, allocates the
// outputs, calls the C ABI.  What Python needs for that is most of such a call: advantages of 128 x 8 rollouts 11.4 us
// a call through ctypes and torch.empty, now 6.6 (the kernel takes 5.7); alignment of short rows 13.3 and 9.3.
//
// A function here returns None for anything it does not take as it is (no plain torch.Tensor, another dtype, not
// contiguous, not on a GPU, any exception): the caller then goes through the Python path, whose checks and errors are
// the ones that count.
#define PY_SSIZE_T_CLEAN
#include <Python.h>
#include <ATen/core/Tensor.h>
#include <ATen/ops/empty.h>
#include <torch/csrc/autograd/python_variable.h>

#include "../../include/mrl.h"

namespace {

// A tensor argument: pointer of a plain contiguous GPU tensor of the dtype; None -> nullptr if allowed.
bool tensor_arg(PyObject* o, at::ScalarType type, bool optional, void** ptr) {
  if (o == Py_None) { *ptr = nullptr; return optional; }
  if (!THPVariable_CheckExact(o)) return false;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.is_cuda() || t.scalar_type() != type || !t.is_contiguous()) return false;
  *ptr = const_cast<void*>(t.const_data_ptr());
  return true;
}

bool int_arg(PyObject* o, int64_t* v) {
  if (!PyLong_CheckExact(o)) return false;
  *v = PyLong_AsLongLong(o);
  if (*v == -1 && PyErr_Occurred()) { PyErr_Clear(); return false; }
  return true;
}
bool int32_arg(PyObject* o, int32_t* v) {
  int64_t w;
  if (!int_arg(o, &w) || w < INT32_MIN || w > INT32_MAX) return false;
  *v = (int32_t)w;
  return true;
}
bool float_arg(PyObject* o, float* v) {
  if (!PyFloat_CheckExact(o)) return false;
  *v = (float)PyFloat_AS_DOUBLE(o);
  return true;
}

at::Tensor new_like(const at::Tensor& t, at::IntArrayRef sizes, at::ScalarType type) {
  return at::empty(sizes, t.options().dtype(type).requires_grad(false));
}

// (rewards, group_id, G, in_stats, scored, is_own, mode, eps_norm, ddof, mix_alpha, neg_thresh, pos_thresh, baseline_shift, stream)
// -> (status, adv, mean, std, flags) or None
PyObject* advantages(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    void *rewards, *group, *in_stats, *scored, *own, *shift;
    int32_t G, mode, ddof;
    float eps, mix, neg, pos;
    int64_t stream;
    if (n != 14 || !tensor_arg(a[0], at::kFloat, false, &rewards) || !tensor_arg(a[1], at::kInt, false, &group) || !int32_arg(a[2], &G) ||
        !tensor_arg(a[3], at::kByte, true, &in_stats) || !tensor_arg(a[4], at::kByte, true, &scored) ||
        !tensor_arg(a[5], at::kByte, true, &own) || !int32_arg(a[6], &mode) || !float_arg(a[7], &eps) || !int32_arg(a[8], &ddof) ||
        !float_arg(a[9], &mix) || !float_arg(a[10], &neg) || !float_arg(a[11], &pos) || !tensor_arg(a[12], at::kFloat, true, &shift) ||
        !int_arg(a[13], &stream) || G <= 0 || (shift != nullptr && THPVariable_Unpack(a[12]).numel() != G))
      Py_RETURN_NONE;
    const at::Tensor& r = THPVariable_Unpack(a[0]);
    const int64_t B = r.numel();
    if (B == 0) Py_RETURN_NONE;
    at::Tensor adv = new_like(r, {B}, at::kFloat), mean = new_like(r, {G}, at::kFloat), std = new_like(r, {G}, at::kFloat);
    at::Tensor flags = new_like(r, {G}, at::kByte);
    // (whatever may throw stands before the GIL is given up: the handler below needs it)
    float *const adv_ptr = static_cast<float*>(adv.mutable_data_ptr()), *const mean_ptr = static_cast<float*>(mean.mutable_data_ptr());
    float* const std_ptr = static_cast<float*>(std.mutable_data_ptr());
    uint8_t* const flags_ptr = static_cast<uint8_t*>(flags.mutable_data_ptr());
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = mrl_group_advantages(static_cast<float*>(rewards), static_cast<int32_t*>(group), static_cast<uint8_t*>(in_stats),
                              static_cast<uint8_t*>(scored), static_cast<uint8_t*>(own), static_cast<float*>(shift), B, G, mode, eps, ddof,
                              mix, neg, pos, adv_ptr, mean_ptr, std_ptr, flags_ptr, reinterpret_cast<void*>(stream));
    Py_END_ALLOW_THREADS
    return Py_BuildValue("(iNNNN)", rc, THPVariable_Wrap(std::move(adv)), THPVariable_Wrap(std::move(mean)),
                         THPVariable_Wrap(std::move(std)), THPVariable_Wrap(std::move(flags)));
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// (src_logp, src_mask, src_word_map, src_map_len, tgt_mask, tgt_word_map, tgt_map_len, max_words, ignore_value, want_bad_count, stream)
// -> (status, out, bad or None) or None
PyObject* align(PyObject*, PyObject* const* a, Py_ssize_t n) {
  try {
    void* p[7];
    static const at::ScalarType types[7] = {at::kFloat, at::kByte, at::kInt, at::kInt, at::kByte, at::kInt, at::kInt};
    int32_t words;
    float ignore;
    int64_t stream;
    if (n != 11) Py_RETURN_NONE;
    for (int i = 0; i < 7; ++i)
      if (!tensor_arg(a[i], types[i], false, &p[i])) Py_RETURN_NONE;
    if (!int32_arg(a[7], &words) || !float_arg(a[8], &ignore) || (a[9] != Py_True && a[9] != Py_False) || !int_arg(a[10], &stream))
      Py_RETURN_NONE;
    const at::Tensor &src = THPVariable_Unpack(a[0]), &tgt = THPVariable_Unpack(a[4]);
    if (src.dim() != 2 || tgt.dim() < 2 || src.size(1) > INT32_MAX || tgt.size(1) > INT32_MAX || src.numel() == 0 || tgt.numel() == 0)
      Py_RETURN_NONE;
    const int64_t B = src.size(0), S_src = src.size(1), S_tgt = tgt.size(1);
    at::Tensor out = new_like(src, {B, S_tgt}, at::kFloat), bad;
    if (a[9] == Py_True) bad = new_like(src, {1}, at::kLong);
    float* const out_ptr = static_cast<float*>(out.mutable_data_ptr());
    int64_t* const bad_ptr = bad.defined() ? static_cast<int64_t*>(bad.mutable_data_ptr()) : nullptr;
    int rc;
    Py_BEGIN_ALLOW_THREADS
    rc = mrl_thl_word_align(static_cast<float*>(p[0]), static_cast<uint8_t*>(p[1]), static_cast<int32_t*>(p[2]), static_cast<int32_t*>(p[3]),
                            static_cast<uint8_t*>(p[4]), static_cast<int32_t*>(p[5]), static_cast<int32_t*>(p[6]), B, (int32_t)S_src,
                            (int32_t)S_tgt, words, ignore, out_ptr, bad_ptr, reinterpret_cast<void*>(stream));
    Py_END_ALLOW_THREADS
    Py_INCREF(Py_None);
    PyObject* second = Py_None;
    if (bad.defined()) { Py_DECREF(Py_None); second = THPVariable_Wrap(std::move(bad)); }
    return Py_BuildValue("(iNN)", rc, THPVariable_Wrap(std::move(out)), second);
  } catch (...) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

PyMethodDef methods[] = {
    {"advantages", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(advantages)), METH_FASTCALL, nullptr},
    {"align", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(align)), METH_FASTCALL, nullptr},
    {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "mrl_host", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit_mrl_host() {
  PyObject* m = PyModule_Create(&module);
  // (the torch whose C++ interface this was compiled against: the caller compares before the first use)
  if (m != nullptr && PyModule_AddStringConstant(m, "torch_version", MRL_TORCH_VERSION) != 0) Py_CLEAR(m);
  return m;
}
