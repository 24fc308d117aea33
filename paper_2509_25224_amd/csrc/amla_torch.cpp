// What amla.amla_decode does between its arguments and the C ABI, as one native call: the checks, the outputs, the workspace, amla_decode().
// A call of the smallest kernels takes the GPU less time than this took in Python (a call with two launches 15.2 us of host work, 7.1 of them
// the launches themselves, 4.6 three allocations by way of Python's argument parser; 7.7 now, with one launch 9.5 before and 4.1 now).
#include <c10/hip/HIPStream.h>
#include <torch/csrc/Exceptions.h>
#include <torch/csrc/autograd/python_variable.h>
#include <torch/extension.h>

#include "amla.h"

namespace {

[[noreturn]] void refuse(PyObject* kind, const char* why) {
  PyErr_SetString(kind, why);
  throw python_error();
}

bool given(PyObject* o) { return o != Py_None; }

// (what reading `attribute` of another object raises)
const at::Tensor& tensor(PyObject* o, const char* attribute) {
  if (THPVariable_Check(o)) return THPVariable_Unpack(o);
  PyErr_Format(PyExc_AttributeError, "'%.200s' object has no attribute '%s': a torch.Tensor is wanted", Py_TYPE(o)->tp_name, attribute);
  throw python_error();
}

int32_t int32(PyObject* o) {   // (as a ctypes field takes it)
  const unsigned long v = PyLong_AsUnsignedLongMask(o);
  if (v == (unsigned long)-1 && PyErr_Occurred()) throw python_error();
  return (int32_t)v;
}

float scale_of(PyObject* o) {   // (as a ctypes argument takes it)
  const double v = PyFloat_AsDouble(o);
  if (v != -1.0 || !PyErr_Occurred()) return (float)v;
  PyErr_Clear();
  THPObjectPtr ctypes(PyImport_ImportModule("ctypes")), error(ctypes ? PyObject_GetAttrString(ctypes.get(), "ArgumentError") : nullptr);
  if (error) PyErr_SetString(error.get(), "softmax_scale: a float is wanted");
  throw python_error();
}

bool usable(const at::Tensor& t, at::ScalarType type) { return t.is_cuda() && t.is_contiguous() && t.scalar_type() == type; }

void sized(const at::Tensor& t, int64_t n) {
  if (t.dim() != n) refuse(PyExc_ValueError, "q has four dimensions, kv_cache three");
}

// decode(q, kv_cache, block_table, seqlens, softmax_scale, out, lse, variant, num_splits, flags, workspace, want_lse, q_lens)
// -> (out, lse, status)
PyObject* decode(PyObject*, PyObject* const* args, Py_ssize_t n_args) {
  HANDLE_TH_ERRORS
  if (n_args != 13) refuse(PyExc_TypeError, "13 arguments are wanted");
  auto input = [&](int k, at::ScalarType type) -> const at::Tensor& {
    const at::Tensor& t = tensor(args[k], "is_cuda");
    if (!usable(t, type)) refuse(PyExc_ValueError, "inputs must be contiguous CUDA tensors of the documented dtypes");
    return t;
  };
  const at::Tensor& q = input(0, at::kBFloat16);
  const at::Tensor& kv = input(1, at::kBFloat16);
  const at::Tensor& table = input(2, at::kInt);
  const at::Tensor& seqlens = input(3, at::kInt);
  sized(q, 4);
  sized(kv, 3);
  const int64_t batch = q.size(0), s_q = q.size(1), heads = q.size(2);
  if (table.size(0) != batch || seqlens.size(0) != batch) refuse(PyExc_ValueError, "block_table / seqlens batch mismatch");
  if (kv.size(2) != q.size(3)) refuse(PyExc_ValueError, "q and kv_cache row widths differ");
  const bool has_q_lens = given(args[12]);
  if (has_q_lens) {
    const at::Tensor& t = tensor(args[12], "is_cuda");
    if (!usable(t, at::kInt) || t.dim() != 1 || t.size(0) != batch)
      refuse(PyExc_ValueError, "q_lens must be a contiguous int32 CUDA tensor of shape [batch]");
  }
  amla_desc d = {};
  d.batch = (int32_t)batch;
  d.s_q = (int32_t)s_q;
  d.num_heads = (int32_t)heads;
  d.d_qk = (int32_t)q.size(3);
  d.d_v = 512;
  d.block_size = (int32_t)kv.size(1);
  d.num_blocks = (int32_t)kv.size(0);
  d.max_blocks_per_seq = (int32_t)table.size(1);
  d.variant = int32(args[7]);
  d.num_splits = int32(args[8]);
  d.flags = int32(args[9]);
  d.stream = c10::hip::getCurrentHIPStream(q.device().index()).stream();
  d.q_lens = has_q_lens ? static_cast<const int32_t*>(tensor(args[12], "data_ptr").data_ptr()) : nullptr;

  const at::Tensor out = given(args[5]) ? tensor(args[5], "data_ptr") : at::empty({batch, s_q, heads, 512}, q.options());
  at::Tensor lse, workspace;
  if (given(args[6])) {
    lse = tensor(args[6], "data_ptr");
  } else {
    const int want_lse = PyObject_IsTrue(args[11]);
    if (want_lse < 0) throw python_error();
    if (want_lse) lse = at::empty({batch, s_q, heads}, q.options().dtype(at::kFloat));
  }
  if (given(args[10])) workspace = tensor(args[10], "data_ptr");
  const size_t need = amla_workspace_bytes(&d);
  if (need > 0 && (!workspace.defined() || workspace.nbytes() < need)) workspace = at::empty({(int64_t)need}, q.options().dtype(at::kByte));
  if (workspace.defined()) {
    d.workspace = workspace.data_ptr();
    d.workspace_bytes = workspace.nbytes();
  }
  const void *q_at = q.data_ptr(), *kv_at = kv.data_ptr();
  const int32_t *table_at = static_cast<const int32_t*>(table.data_ptr()), *seqlens_at = static_cast<const int32_t*>(seqlens.data_ptr());
  void* const out_at = out.data_ptr();
  float* const lse_at = lse.defined() ? static_cast<float*>(lse.data_ptr()) : nullptr;
  const float scale = scale_of(args[4]);
  int status;
  {
    pybind11::gil_scoped_release others_may_run;
    status = amla_decode(q_at, kv_at, table_at, seqlens_at, scale, out_at, lse_at, &d);
  }
  THPObjectPtr out_obj(THPVariable_Wrap(out)), lse_obj(lse.defined() ? THPVariable_Wrap(lse) : (Py_INCREF(Py_None), Py_None));
  if (!out_obj || !lse_obj) throw python_error();
  return Py_BuildValue("(OOi)", out_obj.get(), lse_obj.get(), status);
  END_HANDLE_TH_ERRORS
}

PyMethodDef kMethods[] = {{"decode", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)()>(decode)), METH_FASTCALL, nullptr},
                          {nullptr, nullptr, 0, nullptr}};
PyModuleDef kModule = {PyModuleDef_HEAD_INIT, "_amla_torch", nullptr, -1, kMethods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__amla_torch(void) { return PyModule_Create(&kModule); }
