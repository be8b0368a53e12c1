// The two linear calls of binding.py from tensors to the C ABI in one step of native code.  A one-row call takes the GPU 4.8 us and
// took Python 6.3 to marshal (a method call per data pointer, contiguity, type and size, ctypes' conversions): calls in a row 6.34 us each, 5.35 so.
// Only the plain case is handled: dense tensors that are exactly torch.Tensor, on the GPU, as the call wants them.  Anything else (a subclass, a
// wrapper without storage, a function mode, a wrong type or stride, a failed allocation) returns None, and binding.py's own path, which decides what is
// accepted and raises, takes the call.
#include <Python.h>

#include <ATen/ATen.h>
#include <ATen/PythonTorchFunctionTLS.h>
#include <torch/csrc/autograd/python_variable.h>

#include <exception>

namespace {

using PerChannel = int (*)(const void*, int64_t, const void*, const void*, void*, int32_t*, int64_t, int64_t, int64_t, void*, size_t, void*);
using PerGroup = int (*)(const void*, int64_t, const void*, const int8_t*, const void*, int, int, void*, int32_t*, int64_t, int64_t, int64_t, void*,
                         size_t, void*);
PerChannel per_channel = nullptr;
PerGroup per_group = nullptr;

const at::Tensor* plain(PyObject* o, at::ScalarType type) {
  if (!THPVariable_CheckExact(o)) return nullptr;
  const at::Tensor& t = THPVariable_Unpack(o);
  if (!t.defined() || !t.has_storage() || !t.is_cuda() || t.layout() != at::kStrided || t.scalar_type() != type ||
      t.unsafeGetTensorImpl()->is_python_dispatch())
    return nullptr;
  return &t;
}
const at::Tensor* dense(PyObject* o, at::ScalarType type) {
  const at::Tensor* t = plain(o, type);
  return t && t->is_contiguous() ? t : nullptr;
}

// linear(a_fp16, w_packed, s_g or None, s_w, workspace, y or None, acc_out or None, group, sg_max, stream)
// -> the output, an error code, or None: not a plain call
PyObject* linear(PyObject*, PyObject* const* args, Py_ssize_t n) {
  if (n != 10) Py_RETURN_NONE;
  const bool grouped = args[2] != Py_None;
  if (!(grouped ? per_group != nullptr : per_channel != nullptr)) Py_RETURN_NONE;
  try {
    if (at::impl::PythonTorchFunctionTLS::stack_len() > 0) Py_RETURN_NONE;
    const at::Tensor* a = plain(args[0], at::kHalf);
    const at::Tensor* w = dense(args[1], at::kByte);
    const at::Tensor* s_g = grouped ? dense(args[2], at::kChar) : nullptr;
    const at::Tensor* s_w = dense(args[3], at::kHalf);
    const at::Tensor* ws = dense(args[4], at::kByte);
    const at::Tensor* acc = args[6] == Py_None ? nullptr : dense(args[6], at::kInt);
    if (!a || !w || !s_w || !ws || (grouped && !s_g) || (args[6] != Py_None && !acc) || a->dim() != 2 || s_w->dim() < 1 || a->stride(1) != 1)
      Py_RETURN_NONE;
    const int64_t M = a->size(0), K = a->size(1), N = s_w->size(0);
    const int64_t lda = M > 1 || a->stride(0) > K ? a->stride(0) : K;
    const long group = PyLong_AsLong(args[7]), sg_max = PyLong_AsLong(args[8]);
    void* const stream = PyLong_AsVoidPtr(args[9]);
    if (PyErr_Occurred() || group != (int)group || sg_max != (int)sg_max) {
      PyErr_Clear();
      Py_RETURN_NONE;
    }
    at::Tensor made;
    const at::Tensor* y = nullptr;
    if (args[5] == Py_None) {
      made = at::empty({M, N}, a->options());
      y = &made;
    } else {
      y = dense(args[5], at::kHalf);
    }
    if (!y) Py_RETURN_NONE;
    void *pa = a->data_ptr(), *pw = w->data_ptr(), *ps = s_w->data_ptr(), *py = y->data_ptr(), *pws = ws->data_ptr();
    const int8_t* pg = grouped ? static_cast<const int8_t*>(s_g->data_ptr()) : nullptr;
    int32_t* pacc = acc ? static_cast<int32_t*>(acc->data_ptr()) : nullptr;
    const size_t bytes = static_cast<size_t>(ws->numel());
    int rc;
    Py_BEGIN_ALLOW_THREADS;  // (as ctypes does)
    rc = grouped ? per_group(pa, lda, pw, pg, ps, (int)group, (int)sg_max, py, pacc, M, N, K, pws, bytes, stream)
                 : per_channel(pa, lda, pw, ps, py, pacc, M, N, K, pws, bytes, stream);
    Py_END_ALLOW_THREADS;
    if (rc != 0) return PyLong_FromLong(rc);
    if (args[5] != Py_None) {
      Py_INCREF(args[5]);
      return args[5];
    }
    return THPVariable_Wrap(made);
  } catch (const std::exception&) {
    PyErr_Clear();
    Py_RETURN_NONE;
  }
}

// bind(address of qqq_linear_w4a8_perchannel, of qqq_linear_w4a8_pergroup)
PyObject* bind(PyObject*, PyObject* args) {
  unsigned long long pc = 0, pg = 0;
  if (!PyArg_ParseTuple(args, "KK", &pc, &pg)) return nullptr;
  per_channel = reinterpret_cast<PerChannel>(static_cast<uintptr_t>(pc));
  per_group = reinterpret_cast<PerGroup>(static_cast<uintptr_t>(pg));
  Py_RETURN_NONE;
}

PyMethodDef methods[] = {{"linear", reinterpret_cast<PyCFunction>(reinterpret_cast<void (*)(void)>(linear)), METH_FASTCALL, nullptr},
                         {"bind", bind, METH_VARARGS, nullptr},
                         {nullptr, nullptr, 0, nullptr}};
PyModuleDef module = {PyModuleDef_HEAD_INIT, "_qqq_call", nullptr, -1, methods, nullptr, nullptr, nullptr, nullptr};

}  // namespace

PyMODINIT_FUNC PyInit__qqq_call(void) { return PyModule_Create(&module); }
